"""Python front-end of the gfx950 D3Q19 BGK library.

PyTorch provides device memory and the stream; every step of the solver --
initialisation, the fused stream-collide update, macroscopic fields, FP64
reductions, and the adjoint -- runs in the HIP kernels behind the C ABI of
include/lbm.h.  Shapes are (nz, ny, nx); fields are [nz, ny, nx] and
[3, nz, ny, nx]; populations [19, nz, ny, x_stride] in the interface order.
"""
import ctypes
import math

import torch

from . import _abi as A

STORAGE = {"f32": A.LBM_F32, "f16": A.LBM_F16, "bf16": A.LBM_BF16, "f64": A.LBM_F64,
           "f32x": A.LBM_F32X}
EQUILIBRIUM = {"qian": A.LBM_EQ_QIAN, "incompressible": A.LBM_EQ_INCOMPRESSIBLE}
TORCH_DTYPE = {A.LBM_F32: torch.float32, A.LBM_F16: torch.float16,
               A.LBM_BF16: torch.bfloat16, A.LBM_F64: torch.float64, A.LBM_F32X: torch.float32}


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _aligned(t, what):
    if t.data_ptr() % 256:
        raise ValueError(f"{what} must be 256-byte aligned")
    return t


def _as_field(x, shape, dtype, device, what):
    """A contiguous device tensor of the given shape and dtype (a copy when
    the caller's tensor differs); None stays None."""
    if x is None:
        return None
    t = torch.as_tensor(x)
    if tuple(t.shape) != tuple(shape):
        raise ValueError(f"{what} must have shape {tuple(shape)}, got {tuple(t.shape)}")
    return t.to(device=device, dtype=dtype).contiguous()


class LBM:
    """One D3Q19 BGK simulation on a periodic box (walls and obstacles are
    solid flag bits).  ``storage`` in {'f32', 'f16', 'bf16', 'f64', 'f32x'}
    ('f32x': FP32 storage with FP64 collision arithmetic).  ``wall_u``: the
    velocity of the cells flagged solid + moving (bit 2); ``equilibrium``:
    'qian' (u = j/rho) or 'incompressible' (He-Luo, u = j/rho0);
    ``obstacle_kernel=1`` selects the split design (a separate bounce-back
    kernel before each step) instead of the fused solid markers;
    ``steps_per_pass=2`` runs pairs of steps as one temporally blocked pass
    (same results, bit for bit); ``steps_per_pass="auto"`` does so where pairs
    are faster (boxes up to about 32^3 cells; from 64^3 in FP32, if not flat or
    narrow, and FP64, 74^3 in 16 bits, 102^3 in F32X) and runs single steps
    elsewhere."""

    def __init__(self, shape, tau, force=(0.0, 0.0, 0.0), storage="f32", flags=None, u0=None,
                 rho0=None, f16_scale_log2=0, x_align=0, device="cuda", wall_u=(0.0, 0.0, 0.0),
                 equilibrium="qian", obstacle_kernel=0, steps_per_pass=0):
        self.shape = tuple(int(s) for s in shape)
        if len(self.shape) != 3:
            raise ValueError("shape must be (nz, ny, nx)")
        self.storage = STORAGE[storage] if isinstance(storage, str) else int(storage)
        self.dtype = TORCH_DTYPE[self.storage]
        self.device = torch.device(device)
        if self.device.type != "cuda":
            raise ValueError("the solver runs on a GPU device")
        if self.device.index is None:
            self.device = torch.device("cuda", torch.cuda.current_device())
        self.tau = float(tau)
        self.force = tuple(float(f) for f in force)
        self.wall_u = tuple(float(v) for v in wall_u)
        self.equilibrium = EQUILIBRIUM[equilibrium] if isinstance(equilibrium, str) \
            else int(equilibrium)
        self.params = A.params(self.shape, tau, self.force, self.storage, f16_scale_log2, x_align,
                               self.wall_u, self.equilibrium, obstacle_kernel, steps_per_pass)
        xs, ds, gb, sb, ab = A.lbm_query(self.params)
        self.x_stride, self.dir_stride = xs, ds
        self.grid_bytes, self.adj_partials_bytes = gb, ab
        nz, ny, nx = self.shape
        self.flags = _as_field(flags, self.shape, torch.uint8, self.device, "flags")
        self.rho0 = _as_field(rho0, self.shape, torch.float32, self.device, "rho0")
        self.u0 = _as_field(u0, (3,) + self.shape, torch.float32, self.device, "u0")
        self.grids = [_aligned(torch.empty(gb, dtype=torch.uint8, device=self.device), "grid")
                      for _ in range(2)]
        self.scratch = _aligned(torch.empty(sb, dtype=torch.uint8, device=self.device), "scratch")
        self.stream = torch.cuda.current_stream(self.device)
        self.ctx = A.lbm_init(self.params, _ptr(self.grids[0]), _ptr(self.grids[1]),
                              _ptr(self.flags), _ptr(self.scratch), _ptr(self.rho0),
                              _ptr(self.u0), ctypes.c_void_p(self.stream.cuda_stream))

    # -- state --------------------------------------------------------------
    @property
    def t(self):
        return A.lbm_time(self.ctx)

    @property
    def current(self):
        return A.lbm_current(self.ctx)

    def grid_view(self, buf, dtype=None):
        """A grid-layout buffer viewed as [19, nz, ny, x_stride] (the direction
        arrays dir_stride elements apart): a raw byte buffer in the storage
        dtype (or `dtype`), or a typed buffer (e.g. an FP32 adjoint grid) as is."""
        nz, ny, _ = self.shape
        t = buf.view(dtype or self.dtype) if buf.dtype == torch.uint8 else buf
        xs = self.x_stride
        return torch.as_strided(t, (19, nz, ny, xs), (self.dir_stride, ny * xs, xs, 1))

    def populations(self):
        """View of the current grid: offsets g = f* - w (FP16: 2^s g)."""
        return self.grid_view(self.grids[self.current])

    def new_grid(self):
        return _aligned(torch.empty(self.grid_bytes, dtype=torch.uint8, device=self.device), "grid")

    # -- the hot path -------------------------------------------------------
    def step(self, n=1):
        A.lbm_step(self.ctx, n)
        return self

    def step_from(self, src, dst):
        A.lbm_step_from(self.ctx, _ptr(_aligned(src, "src")), _ptr(_aligned(dst, "dst")))

    def step2_from(self, src, mid, dst):
        """Two steps from ``src`` in one fused pass: ``mid`` gets the first
        state, ``dst`` the second (FP32 storage)."""
        A.lbm_step2_from(self.ctx, _ptr(_aligned(src, "src")), _ptr(_aligned(mid, "mid")),
                         _ptr(_aligned(dst, "dst")))

    def macroscopics(self, f64=False):
        dt = torch.float64 if f64 else torch.float32
        rho = torch.empty(self.shape, dtype=dt, device=self.device)
        u = torch.empty((3,) + self.shape, dtype=dt, device=self.device)
        (A.lbm_macroscopics_f64 if f64 else A.lbm_macroscopics)(self.ctx, _ptr(rho), _ptr(u))
        return rho, u

    def reduce(self):
        """Device tensor (float64, 5): mass, momentum x/y/z, kinetic energy."""
        out = torch.empty(5, dtype=torch.float64, device=self.device)
        A.lbm_reduce(self.ctx, _ptr(out))
        return out

    # -- checkpoint / resume --------------------------------------------------
    def save(self, dst=None):
        dst = self.new_grid() if dst is None else _aligned(dst, "dst")
        A.lbm_save(self.ctx, _ptr(dst))
        return dst

    def restore(self, src, t):
        A.lbm_restore(self.ctx, _ptr(src), t)

    def refresh_solids(self):
        """Rewrite the solid-cell markers of the current grid (after
        populations were written into it directly) and the two-step pass's
        link mask (after the flags were changed in place)."""
        A.lbm_refresh_solids(self.ctx)

    def set_current(self, parity, t):
        A.lbm_set_current(self.ctx, parity, t)

    def pull_copy(self, src, dst):
        """Pull-copy probe: dst_i(x) = src_i(x - c_i) over this grid layout
        (periodic, no geometry, no collision), launched like the step."""
        A.lbm_pull_copy(self.ctx, _ptr(_aligned(src, "src")), _ptr(_aligned(dst, "dst")))
        return self

    def use_graphs(self, steps_per_graph):
        """Replay HIP graphs of `steps_per_graph` (even) captured steps in
        step() -- for launch-bound small grids; 0 turns it off."""
        A.lbm_use_graphs(self.ctx, steps_per_graph)
        return self

    def close(self):
        if getattr(self, "ctx", None):
            A.lbm_destroy(self.ctx)
            self.ctx = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def stream_copy(dst, src, stream=None):
    """STREAM copy dst = src of whole tensors on the GPU (bandwidth probe)."""
    if dst.numel() * dst.element_size() != src.numel() * src.element_size():
        raise ValueError("size mismatch")
    s = torch.cuda.current_stream() if stream is None else stream
    A.lbm_stream_copy(_ptr(_aligned(dst, "dst")), _ptr(_aligned(src, "src")),
                      src.numel() * src.element_size(), ctypes.c_void_p(s.cuda_stream))


def copy_probe(dst, src, vec_per_thread=1, nontemporal=False, blocks=0, stream=None):
    """A variant of the copy dst = src for the bandwidth sweep (16-byte
    elements per thread, non-temporal accesses, grid-stride block count)."""
    if dst.numel() * dst.element_size() != src.numel() * src.element_size():
        raise ValueError("size mismatch")
    s = torch.cuda.current_stream() if stream is None else stream
    A.lbm_copy_probe(_ptr(_aligned(dst, "dst")), _ptr(_aligned(src, "src")),
                     src.numel() * src.element_size(), vec_per_thread, int(bool(nontemporal)),
                     blocks, ctypes.c_void_p(s.cuda_stream))


# The rollout steps in fused pairs, forward and in the recomputation (the same
# states bit for bit), where the library finds them faster (lbm_pairs: us a step,
# single / pairs, 24^3 3.4 / 2.8, 64^3 7.4 / 7.1, 128^3 57 / 41, 256^3 457 / 271), on
# boxes of at least this many cells.
FUSED_RECOMPUTE_MIN_CELLS = 0

# The reverse sweep runs in pairs of steps from this many cells on.  Measured, us a
# step, single / pairs: 48^3 7.4 / 9.0, 64^3 11.0 / 10.4, 100^3 38 / 30, 128^3 64 /
# 43, 256^3 501 / 327.
ADJOINT_PAIRS_MIN_CELLS = 1 << 18

# How much of the device's memory a rollout may take for the moments that its
# forward sweep keeps beyond the last segment's (288 GB: 4.5 GB, about 140 steps of
# 128^3).  Kept, a step's moments cost the pass that runs anyway 5 us at 128^3;
# recomputed, half of a 95 us pass.  Rollouts that wait for their backward together
# take no more than half of the memory in this way.
KEPT_MOMENTS_SHARE = 1 / 64


class _Rollout(torch.autograd.Function):
    """(rho_T, u_T) after `steps` updates from f*(0) = f^eq(1, u0) under the
    body force g; backward runs the hand-written adjoint kernels with forward
    checkpoints every k steps.  The reverse step n needs of the state f(n) its
    moments only (16 B per cell and step); the forward sweep stores them for
    the last segment, the others are recomputed from their checkpoints."""

    @staticmethod
    def forward(ctx, u0, g, steps, tau, flags, k, wall_u, equilibrium, steps_per_pass, need_grad):
        force = [float(v) for v in g.detach().double().cpu().tolist()]
        cells = math.prod(u0.shape[1:])
        fused = cells >= FUSED_RECOMPUTE_MIN_CELLS and A.lbm_pairs(A.params(u0.shape[1:], tau, force))
        schedule = steps_per_pass
        if schedule in (-1, 0, 1):  # automatic also for the link mask, which the reverse pairs read
            reverse_pairs = need_grad and cells >= ADJOINT_PAIRS_MIN_CELLS
            schedule = 2 if fused else (-1 if reverse_pairs else schedule)
        sim = LBM(u0.shape[1:], tau, force, "f32", flags=flags, u0=u0.detach(), device=u0.device,
                  x_align=_Rollout.row_align(u0.shape[1:]), wall_u=wall_u, equilibrium=equilibrium,
                  steps_per_pass=schedule)
        if not need_grad:
            sim.step(steps)
            return sim.macroscopics()
        pairs = fused or steps_per_pass == 2
        starts = range(0, steps, k)  # the segments of k steps
        last = len(starts) - 1
        first = _Rollout.first_kept(sim, steps, k)
        cur, spare, tmp = sim.grids[0], None, _Rollout.second_grid(sim, min(k, steps), pairs)
        ckpts, moms = [], []
        for s, t in enumerate(starts):
            if s < first:
                ckpts.append(cur)
            if s + 1 < first:
                dst = sim.new_grid()
            elif first == 0:
                dst = sim.grids[1 - s % 2]
            elif (last - s) % 2 == 0:
                dst = sim.grids[1]
            else:
                dst = spare = sim.new_grid() if spare is None else spare
            n = min(k, steps - t)
            moms.append(None if s < first else _Rollout.moments(sim, n))
            A.lbm_segment(sim.ctx, _ptr(cur), _ptr(tmp), _ptr(dst), n, pairs, _ptr(moms[s]), True)
            cur = dst
        sim.set_current(0 if cur is sim.grids[0] else 1, steps)
        rho, u = sim.macroscopics()
        ctx.sim, ctx.ckpts, ctx.steps, ctx.k = sim, ckpts, steps, k
        ctx.moms, ctx.fused = moms, fused
        ctx.g_meta = (g.dtype, g.device)
        return rho, u

    @staticmethod
    def row_align(shape):
        """Rows padded to 16 bytes only, where two such grids stay in the 256 MB cache
        and the rows span a sixteenth fewer of the 128-byte lines in which it is
        read (24 steps and back: 72 x 80 x 100 1.19 -> 1.11 ms, 100^3 1.90 -> 1.67,
        120^3 3.25 -> 2.52; 90^3, where 4% are saved, 1.35 -> 1.40).  Grids streamed
        from memory want their rows on 64-byte sectors (a reverse step of 200^3 314
        us padded, 355 tight) and keep the default."""
        nz, ny, nx = shape
        tight, lines = -(-nx // 4) * 4, -(-nx // 32) * 32
        return 4 if 16 * tight <= 15 * lines and 2 * 76 * nz * ny * tight <= 256 << 20 else 0

    @staticmethod
    def first_kept(sim, steps, k):
        """The first segment whose moments the forward sweep keeps: the last one and
        as many before it as fit in KEPT_MOMENTS_SHARE of the device's memory, if
        half of that memory stays free (blocks that torch holds unused count as
        free).  Else none: the rollout then holds its checkpoints only."""
        last, record = (steps - 1) // k, 16 * sim.dir_stride  # bytes of a step's moments
        least = (steps - last * k) * record
        if last == 0 and least < 1 << 26:  # not worth asking
            return 0
        free, total = torch.cuda.mem_get_info(sim.device)
        room = max(least, int(KEPT_MOMENTS_SHARE * total))
        if free - total // 2 < room:
            free += torch.cuda.memory_reserved(sim.device) - torch.cuda.memory_allocated(sim.device)
        fit = min(room, free - total // 2)
        if fit < least:
            return last + 1
        return min(last, max(0, -((fit // record - steps) // k)))

    @staticmethod
    def second_grid(sim, n, pairs):
        """The other grid of a segment of n steps, unless one pass does."""
        return sim.new_grid() if n > (2 if pairs else 1) else None

    @staticmethod
    def adjoint_pairs(sim):
        """Whether the reverse sweep runs in pairs of steps, paired by their distance
        from the end alone (so that dL/dF, summed pass by pass, does not depend on
        the checkpoints)."""
        return math.prod(sim.shape) >= ADJOINT_PAIRS_MIN_CELLS and A.lbm_adjoint_pairs(sim.ctx)

    @staticmethod
    def moments(sim, n):
        return torch.empty(n * 4 * sim.dir_stride, dtype=torch.float32, device=sim.device)

    @staticmethod
    def backward(ctx, g_rho, g_u):
        """Reverse sweep in pull form: nu^T from the seed at f(T), then nu^n
        from nu^{n+1} at f(n) for n = T-1 .. 1, then dL/du0 from nu^1; the
        moments of the f(n) are recomputed segment by segment from the
        checkpoints, latest segment first."""
        sim, ckpts, moms, steps, k = ctx.sim, ctx.ckpts, ctx.moms, ctx.steps, ctx.k
        dev = sim.device
        nfl = sim.grid_bytes // 4
        nu = [torch.empty(nfl, dtype=torch.float32, device=dev) for _ in range(2)]
        partials = torch.empty(sim.adj_partials_bytes // 8, dtype=torch.float64, device=dev)
        gr = None if g_rho is None else g_rho.to(torch.float32).contiguous()
        gu = None if g_u is None else g_u.to(torch.float32).contiguous()
        record = 4 * sim.dir_stride
        pairs = _Rollout.adjoint_pairs(sim)
        cur, mom, tmp, left = 0, None, None, None  # left: a state that waits for the next pair
        for s in range(len(moms) - 1, -1, -1):
            seed = s == len(moms) - 1
            n = min(k, steps - s * k)
            seg = moms[s]
            if seg is None:
                if mom is None:
                    mom = _Rollout.moments(sim, k)
                    tmp = _Rollout.second_grid(sim, k, ctx.fused)
                elif left is not None:
                    left = left.clone()
                seg = mom
                A.lbm_segment(sim.ctx, _ptr(ckpts[s]), _ptr(tmp), _ptr(sim.grids[1]), n,
                              ctx.fused, _ptr(seg), False)
            if not pairs:
                A.lbm_adjoint_segment(sim.ctx, _ptr(seg), n, seed, _ptr(gr), _ptr(gu),
                                      _ptr(nu[cur]), _ptr(nu[cur ^ 1]), _ptr(partials))
                cur ^= (n - seed) & 1
                continue
            states = [seg[j * record:(j + 1) * record] for j in range(n - 1, -1, -1)]
            if seed:
                A.lbm_adjoint_segment(sim.ctx, _ptr(states.pop(0)), 1, True, _ptr(gr), _ptr(gu),
                                      _ptr(nu[0]), None, _ptr(partials))
            for state in states:
                if left is None:
                    left = state
                    continue
                A.lbm_adjoint_pair(sim.ctx, _ptr(left), _ptr(state), _ptr(nu[cur]),
                                   _ptr(nu[cur ^ 1]), _ptr(partials))
                cur, left = cur ^ 1, None
        if left is not None:
            A.lbm_adjoint_segment(sim.ctx, _ptr(left), 1, False, None, None, _ptr(nu[cur]),
                                  _ptr(nu[cur ^ 1]), _ptr(partials))
            cur ^= 1
        du0 = torch.empty((3,) + sim.shape, dtype=torch.float32, device=dev)
        A.lbm_adjoint_init(sim.ctx, _ptr(nu[cur]), _ptr(sim.rho0), _ptr(sim.u0), _ptr(du0))
        dF = torch.empty(3, dtype=torch.float64, device=dev)
        A.lbm_adjoint_finish_dF(sim.ctx, _ptr(partials), _ptr(dF))
        gdt, gdev = ctx.g_meta
        return (du0, dF.to(device=gdev, dtype=gdt)) + (None,) * 8


def rollout(u0, g, *, steps, tau, flags=None, checkpoint_every=20, wall_u=(0.0, 0.0, 0.0),
            equilibrium="qian", steps_per_pass=0):
    """Differentiable D3Q19 BGK rollout (FP32 storage): returns (rho_T, u_T)
    with gradients for the initial velocity ``u0`` [3, nz, ny, nx] and the
    body-force density ``g`` [3].  Moving walls and the incompressible
    equilibrium are supported (no gradient for the wall velocity).
    ``steps_per_pass=2`` runs the forward sweep in fused pairs of steps on
    every box, not only where they are faster (the same states bit for bit, so
    the same gradients).  The reverse sweep needs 16 B per cell of every state.
    Until its backward a rollout holds two grids of 76 B per cell, those 16 B of
    the last ``checkpoint_every`` steps, of earlier ones up to 1/64 of the device's
    memory, and a grid for every further ``checkpoint_every`` steps, from which the
    others are recomputed; if that left less than half of the memory free, it holds
    the grids only.  (The gradients are the same either way and for any spacing.)"""
    if u0.dim() != 4 or u0.shape[0] != 3:
        raise ValueError("u0 must be [3, nz, ny, nx]")
    if g.numel() != 3:
        raise ValueError("g must have 3 components")
    if steps < 1 or checkpoint_every < 1:
        raise ValueError("steps and checkpoint_every must be >= 1")
    return _Rollout.apply(u0, g.reshape(3), int(steps), float(tau), flags, int(checkpoint_every),
                          tuple(float(v) for v in wall_u), equilibrium, int(steps_per_pass),
                          torch.is_grad_enabled() and (u0.requires_grad or g.requires_grad))
