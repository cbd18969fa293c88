// Program-counter virtual machine: Algorithm 2 of the paper as a HIP interpreter.
//
// One batch member per lane, one lock-step group per 64-lane wavefront.  Per step the group takes the
// smallest block index any of its members waits for, and runs that block's operations for all lanes with
// the writes masked to the members that wait there (the masking style of Section 2).  The top entry of every
// stack is cached (LDS for the variables, a register for the program counter: the fourth optimisation of
// Section 3.2); the entries below it live in global memory as [variable][depth][member], so a push or pop of
// the whole group is one coalesced store or load.  Block and operation records are read through uniform
// indices.  There is no CPU path: without a device the entry point fails.
//
// Programs of up to 64 blocks and 64 operations take pcvm_small_kernel, which keeps all of that in registers and LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <vector>

#include "../../include/pcvm.h"

namespace {

thread_local char g_err[512] = "";
thread_local hipStream_t g_stream = nullptr;

int fail(int code, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

#define PCVM_TRY(expr, code)                                                                    \
    do {                                                                                         \
        hipError_t e_ = (expr);                                                                  \
        if (e_ != hipSuccess) return fail(code, "%s: %s", #expr, hipGetErrorString(e_));         \
    } while (0)

constexpr int kWave = PCVM_GROUP;
constexpr int kWavesPerBlock = 4;

struct VmArgs {
    const pcvm_block* blocks;
    const pcvm_op* ops;
    int n_vars, n_inputs, output_var, n_blocks;
    long batch, batch_pad;  // batch_pad: lanes launched = row pitch of the stacks (one stack column per lane)
    unsigned long long* queue;  // queued runs: index of the next member nobody has taken yet
    int policy;                 // queued runs: PCVM_SCHED_*
    int depth;
    long max_steps;
    const long long* inputs;
    long long* outputs;
    long long* var_stacks;  // [n_vars][depth][batch_pad]
    int* pc_stacks;         // [depth][batch_pad]
    int* trace;
    long trace_capacity;
    unsigned long long* counters;  // steps, active member steps
    int* error;                    // most severe error code seen (most negative)
};

// Minimum over the 64 lanes: rotations inside each row of 16 lanes (DPP, no LDS traffic), then the four
// row minima are read as scalars.
template <int kCtrl>
__device__ __forceinline__ int dpp_move(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, kCtrl, 0xf, 0xf, false);
}
__device__ __forceinline__ int wave_min(int x)
{
    x = min(x, dpp_move<0x128>(x));  // row_ror:8
    x = min(x, dpp_move<0x124>(x));  // row_ror:4
    x = min(x, dpp_move<0x122>(x));  // row_ror:2
    x = min(x, dpp_move<0x121>(x));  // row_ror:1
    return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
               min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

// The block most lanes wait for (the lowest such block on a tie); `halt` if nobody waits.
__device__ __forceinline__ int most_waiting(int pc_top, int halt)
{
    unsigned long long todo = __ballot(pc_top < halt);
    int best = halt, best_count = 0;
    while (todo) {
        const int b = __builtin_amdgcn_readlane(pc_top, (int)__builtin_ctzll(todo));
        const unsigned long long same = __ballot(pc_top == b);
        const int count = __popcll(same);
        if (count > best_count || (count == best_count && b < best)) {
            best = b;
            best_count = count;
        }
        todo &= ~same;
    }
    return best;
}

// y = f(a, b, imm): total functions on 64-bit integers, wrap-around.
__device__ __forceinline__ long long primitive(int fn, long long a, long long b, long long imm)
{
    typedef unsigned long long u64;
    switch (fn) {
    case PCVM_CONST: return imm;
    case PCVM_COPY: return a;
    case PCVM_ADD: return (long long)((u64)a + (u64)b);
    case PCVM_SUB: return (long long)((u64)a - (u64)b);
    case PCVM_MUL: return (long long)((u64)a * (u64)b);
    case PCVM_ADDI: return (long long)((u64)a + (u64)imm);
    case PCVM_MULI: return (long long)((u64)a * (u64)imm);
    case PCVM_LE: return a <= b;
    case PCVM_LT: return a < b;
    case PCVM_EQ: return a == b;
    case PCVM_LEI: return a <= imm;
    case PCVM_EQI: return a == imm;
    case PCVM_MOD: return (b == 0 || b == -1) ? 0 : a % b;
    case PCVM_ANDI: return a & imm;
    case PCVM_SHRI: return a >> (imm & 63);
    default: return 0;
    }
}

// kQueued = false: lane l of group g runs member 64 g + l and nothing else (Algorithm 2 on fixed groups).
// kQueued = true: a lane whose member has halted takes the next member from a global queue, so a group keeps
// all its lanes busy until the batch runs dry - members at the first block of a new execution are batched
// with members deep inside an old one, which is what the program-counter formulation makes possible.
template <bool kQueued>
__global__ __launch_bounds__(kWave* kWavesPerBlock) void pcvm_kernel(VmArgs va)
{
    __shared__ long long s_top[kWavesPerBlock][PCVM_MAX_VARS][kWave];
    __shared__ int s_sp[kWavesPerBlock][PCVM_MAX_VARS][kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const long group = (long)blockIdx.x * kWavesPerBlock + w;
    const long slot = group * kWave + lane;  // this lane's column in the stack arrays
    long member = kQueued ? -1 : slot;
    bool valid = !kQueued && member < va.batch;
    const int halt = va.n_blocks;

    // "PUSH T onto x": a fresh execution has its inputs on the stacks, every other stack empty, and waits at block 0
    auto start_member = [&]() {
        for (int v = 0; v < va.n_vars; ++v) {
            const bool is_input = v < va.n_inputs;
            s_top[w][v][lane] = (is_input && valid) ? va.inputs[(size_t)v * va.batch + member] : 0;
            s_sp[w][v][lane] = is_input ? 1 : 0;
        }
    };
    start_member();
    int pc_top = valid ? 0 : halt;
    int pc_sp = valid ? 1 : 0;
    long steps = 0, member_steps = 0;
    unsigned long long active_steps = 0;
    int my_error = 0;
    // queued runs: the queue was empty when this lane asked, or its member failed - or the lane belongs to a wave of
    // the last workgroup beyond the last group, which has no stack columns and must not take a member
    bool retired = slot >= va.batch_pad;

    for (;;) {
        if (kQueued && pc_sp == 0 && !retired) {
            const long next = (long)atomicAdd(va.queue, 1ull);
            if (next < va.batch) {
                member = next;
                valid = true;
                start_member();
                pc_top = 0;
                pc_sp = 1;
                member_steps = 0;
            } else {
                retired = true;
            }
        }
        if (kQueued && pc_sp > 0 && member_steps >= va.max_steps) {  // this member does not halt: drop it
            my_error = PCVM_E_STEP_LIMIT;
            pc_top = halt;
            pc_sp = 0;
            retired = true;
        }
        // the earliest block anyone waits for (Algorithm 2), or the one most lanes wait for (a scalar either way)
        const int i = (kQueued && va.policy == PCVM_SCHED_MOST_WAITING) ? most_waiting(pc_top, halt) : wave_min(pc_top);
        if (i >= halt) break;
        if (!kQueued && steps >= va.max_steps) {
            my_error = PCVM_E_STEP_LIMIT;
            break;
        }
        const bool A = pc_top == i;  // locally active set
        const pcvm_block blk = va.blocks[i];
        for (int k = 0; k < blk.n_ops; ++k) {
            const pcvm_op op = va.ops[blk.first_op + k];
            long long& top = s_top[w][op.dst][lane];
            int& sp = s_sp[w][op.dst][lane];
            long long* stack = va.var_stacks + (size_t)op.dst * va.depth * va.batch_pad + slot;
            if (op.kind == PCVM_POP) {
                if (A) {
                    if (sp <= 0) {
                        my_error = min(my_error, (int)PCVM_E_STACK_UNDERFLOW);
                    } else {
                        sp -= 1;
                        if (sp >= 1) top = stack[(size_t)(sp - 1) * va.batch_pad];
                    }
                }
                continue;
            }
            const long long o = primitive(op.fn, s_top[w][op.a][lane], s_top[w][op.b][lane], op.imm);
            if (!A) continue;
            if (op.kind == PCVM_PUSH) {
                if (sp >= va.depth) {
                    my_error = min(my_error, (int)PCVM_E_STACK_OVERFLOW);
                } else {
                    if (sp >= 1) stack[(size_t)(sp - 1) * va.batch_pad] = top;  // the old top goes below
                    sp += 1;
                    top = o;
                }
            } else {
                top = o;
            }
        }
        if (A) {
            switch (blk.term) {
            case PCVM_JUMP: pc_top = blk.i; break;
            case PCVM_BRANCH: pc_top = s_top[w][blk.x][lane] != 0 ? blk.i : blk.j; break;
            case PCVM_PUSHJUMP:
                if (pc_sp >= va.depth) {
                    my_error = min(my_error, (int)PCVM_E_STACK_OVERFLOW);
                } else {
                    va.pc_stacks[(size_t)(pc_sp - 1) * va.batch_pad + slot] = blk.j;  // where this frame resumes
                    pc_sp += 1;
                    pc_top = blk.i;  // the callee's entry
                }
                break;
            default:  // PCVM_RETURN
                pc_sp -= 1;
                pc_top = pc_sp >= 1 ? va.pc_stacks[(size_t)(pc_sp - 1) * va.batch_pad + slot] : halt;
                if (kQueued && pc_sp == 0 && !my_error) va.outputs[member] = s_top[w][va.output_var][lane];
                break;
            }
            if (my_error) {  // a member in error stops; the others of its group go on
                pc_top = halt;
                pc_sp = 0;
                retired = true;
            }
        }
        member_steps += 1;
        const unsigned long long amask = __ballot(A);
        if (va.trace && group == 0 && lane == 0 && steps < va.trace_capacity) {
            va.trace[2 * steps] = i;
            va.trace[2 * steps + 1] = __popcll(amask);
        }
        steps += 1;
        active_steps += (unsigned long long)__popcll(amask);
    }

    if (!kQueued && valid) va.outputs[member] = s_top[w][va.output_var][lane];
    if (my_error) atomicMin(va.error, my_error);
    if (lane == 0) {
        atomicAdd(&va.counters[0], (unsigned long long)steps);
        atomicAdd(&va.counters[1], active_steps);
    }
}

// ---- programs of up to 64 blocks and 64 operations ----
//
// A step is a serial chain - choose a block, fetch its record, run its operations one after the other, go on - and a
// batch lasts as long as its longest member, so what bounds it is the latency of a step, not how much a step does
// (fibonacci, 200 000 members in fixed groups: 35 200 steps per group of 4830 ticks each at three groups per SIMD, with the
// records read through the scalar cache and the stacks in global memory).  It is made of round trips to memory and of
// scalar instructions that wait for a vector one, some 50 ticks each.  So
//   * lane k holds operation k and block k, and a record is two v_readlane,
//   * the entries below a top are in a ring of `ring` entries per stack in LDS; only what a deeper push drives out of
//     the ring goes to global memory, and only a pop that reaches below the ring reads it back,
//   * moves, sums, differences and comparisons are straight-line code, as are updates and pushes (an update's push goes
//     to a spare row), jumps, branches and calls; what is rare is out of line,
//   * the block most lanes wait for is found by counting lanes block by block, eight at a time.
// That step takes 2280 ticks (1690 with one group per SIMD).  200 000 members: fibonacci 71.5 -> 33.8 ms in fixed groups,
// 46.6 -> 38.4 queued with MOST_WAITING; collatz_steps 1.62 -> 0.86; binomial (176 408, queued) 6.4 -> 4.7.
constexpr int kSmallMax = 64;

// Operation classes.  Move, add and subtract are one expression, (a & keep) + (b ^ flip) - flip; immediates lie in LDS
// behind the tops and are read as operands that are the same for every lane.
enum : int { kClsMove = 0, kClsAdd = 1, kClsSub = 2, kClsLe = 3, kClsLt = 4, kClsEq = 5, kClsMul = 6, kClsAnd = 7, kClsShr = 8, kClsMod = 9 };
// Packed records, one per lane.  Operations: x = {operand a | operand b << 16} as offsets in 8-byte rows of LDS (variable v:
// 64 v; immediate of operation k: behind the tops, its own cell), y = {dst | class << 4 | b is an immediate << 8 |
// kind << 12 | stack << 16}.  Blocks: x = {first_op | n_ops << 8 | term << 16 | variable << 20}, y = {i | j << 8}.
struct SmallTables {
    unsigned input_stacks;  // bit s: stack s belongs to an input
    unsigned op_x[kSmallMax], op_y[kSmallMax], blk_x[kSmallMax], blk_y[kSmallMax];
    long long imm[kSmallMax];
};

bool small_program(const pcvm_program* p) { return p->n_blocks <= kSmallMax && p->n_ops <= kSmallMax; }

// Returns the number of variables that keep a stack (those that are pushed or popped).
int pack_small(const pcvm_program* p, SmallTables* t)
{
    *t = SmallTables{};
    int stack_of[PCVM_MAX_VARS], n_stacks = 0;
    for (int v = 0; v < PCVM_MAX_VARS; ++v) stack_of[v] = -1;
    for (int o = 0; o < p->n_ops; ++o)
        if (p->ops[o].kind != PCVM_UPDATE && stack_of[p->ops[o].dst] < 0) stack_of[p->ops[o].dst] = n_stacks++;
    for (int o = 0; o < p->n_ops; ++o) {
        const pcvm_op& op = p->ops[o];
        int cls = kClsMove, a = op.a, b = op.b;
        bool imm = false;
        if (op.kind == PCVM_POP) {
            a = b = op.dst;
        } else {
            switch (op.fn) {
            case PCVM_CONST: imm = true; break;
            case PCVM_COPY: b = a; break;
            case PCVM_ADD: cls = kClsAdd; break;
            case PCVM_SUB: cls = kClsSub; break;
            case PCVM_MUL: cls = kClsMul; break;
            case PCVM_ADDI: cls = kClsAdd; imm = true; break;
            case PCVM_MULI: cls = kClsMul; imm = true; break;
            case PCVM_LE: cls = kClsLe; break;
            case PCVM_LT: cls = kClsLt; break;
            case PCVM_EQ: cls = kClsEq; break;
            case PCVM_LEI: cls = kClsLe; imm = true; break;
            case PCVM_EQI: cls = kClsEq; imm = true; break;
            case PCVM_MOD: cls = kClsMod; break;
            case PCVM_ANDI: cls = kClsAnd; imm = true; break;
            default: cls = kClsShr; imm = true; break;  // PCVM_SHRI
            }
        }
        const int stack = stack_of[op.dst] < 0 ? 0 : stack_of[op.dst];
        if (stack_of[op.dst] >= 0 && op.dst < p->n_inputs) t->input_stacks |= 1u << stack;
        const int off_b = imm ? p->n_vars * kWave + o : b * kWave;
        t->op_x[o] = (unsigned)(a * kWave) | (unsigned)off_b << 16;
        t->op_y[o] = (unsigned)(op.dst | cls << 4 | (int)imm << 8 | op.kind << 12 | stack << 16);
        t->imm[o] = op.imm;
    }
    for (int b = 0; b < p->n_blocks; ++b) {
        const pcvm_block& k = p->blocks[b];
        const int first = k.n_ops > 0 ? k.first_op : 0, x = k.term == PCVM_BRANCH ? k.x : 0;
        const int i = k.term == PCVM_RETURN ? 0 : k.i, j = (k.term == PCVM_BRANCH || k.term == PCVM_PUSHJUMP) ? k.j : 0;
        t->blk_x[b] = (unsigned)(first | k.n_ops << 8 | k.term << 16 | x << 20);
        t->blk_y[b] = (unsigned)(i | j << 8);
    }
    return n_stacks;
}

struct SmallArgs {
    const SmallTables* tables;
    int n_stacks;
    int ring;   // entries per stack in LDS, a power of two
    int lanes;  // queued runs: lanes of a group that take members
};

// LDS of a wave, lane by lane: tops [variable], immediates (one cell each, all lanes the same), a spare row, rings
// [stack][entry], stack counts [stack] (entries on the stack | index of the lowest one below the top that is in the ring
// << 16), program counters [entry] and a spare row.
__host__ __device__ inline size_t small_wave_bytes(int n_vars, int n_stacks, int ring)
{
    return ((size_t)n_vars * 8 + 16 + (size_t)(n_stacks > 0 ? n_stacks : 1) * (8 * ring + 4) + (size_t)ring * 4 + 4 + 7) / 8 * 8 * kWave;
}
__device__ __forceinline__ int field(unsigned w, int shift, unsigned mask) { return (int)((w >> shift) & mask); }

template <bool kQueued>
__global__ __launch_bounds__(kWave* kWavesPerBlock) void pcvm_small_kernel(VmArgs va, SmallArgs sm)
{
    typedef unsigned long long u64;
    extern __shared__ __align__(16) unsigned char small_lds[];
    const int lane = threadIdx.x & (kWave - 1), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const long group = (long)blockIdx.x * kWavesPerBlock + w;
    // this lane's column in the stack arrays (queued runs: only lanes that take members have one)
    const long slot = kQueued ? group * sm.lanes + lane : group * kWave + lane;
    if (group * (kQueued ? sm.lanes : kWave) >= va.batch_pad) return;  // waves of the last workgroup beyond the last group
    const int W = sm.ring;
    u64* const rows = reinterpret_cast<u64*>(small_lds + (size_t)w * small_wave_bytes(va.n_vars, sm.n_stacks, W));
    u64* const tops = rows + lane;
    u64* const rings = tops + (va.n_vars + 2) * kWave;  // (the row before the first ring is the spare one)
    const int n_stacks = sm.n_stacks > 0 ? sm.n_stacks : 1;
    unsigned* const counts = reinterpret_cast<unsigned*>(rings - lane + n_stacks * W * kWave) + lane;
    int* const pc_ring = reinterpret_cast<int*>(counts) + (n_stacks + 1) * kWave;  // (spare row in front)
    const unsigned r_opx = sm.tables->op_x[lane], r_opy = sm.tables->op_y[lane];
    const unsigned r_blkx = sm.tables->blk_x[lane], r_blky = sm.tables->blk_y[lane];
    tops[va.n_vars * kWave] = (u64)sm.tables->imm[lane];
    constexpr int kHalt = 255;

    // Queued runs: the first member of a lane is the one of its column, without asking; the queue holds those beyond the last
    // column.  (A lane that asks is one atomic of a wave on one address, and the fewer lanes a group has, the fewer ask
    // together: gcd, 20 000 members in 1000 groups, all members through the queue 0.225 ms, so 0.106; 313 full groups through the
    // queue, interpreter of larger programs, 0.178.)
    long member = slot;
    const bool valid = (!kQueued || lane < sm.lanes) && member < va.batch;
    int pc_sp = 0, pc_low = 0, pc = kHalt;
    long steps = 0, member_start = 0;
    u64 active_steps = 0;
    int my_error = 0;
    bool retired = kQueued && !valid;  // the queue was empty when this lane asked, or its member failed
    bool at_limit = false;
    const bool tracing = !kQueued && va.trace && group == 0;

    // "PUSH T onto x": a fresh execution has its inputs on the stacks, every other stack empty, and waits at block 0
    auto start_member = [&]() __attribute__((always_inline)) {
        for (int v = 0; v < va.n_vars; ++v) tops[v * kWave] = v < va.n_inputs ? (u64)va.inputs[(size_t)v * va.batch + member] : 0ull;
        for (int s = 0; s < sm.n_stacks; ++s) counts[s * kWave] = (sm.tables->input_stacks >> s) & 1u;
        pc = 0;
        pc_sp = 1;
        pc_low = 0;
        member_start = steps;
    };
    if (valid) start_member();

    for (;;) {
        if (kQueued && __ballot(pc == kHalt && !retired)) {
            if (pc == kHalt && !retired) {
                const long next = va.batch_pad + (va.batch_pad < va.batch ? (long)atomicAdd(va.queue, 1ull) : 0);
                if (next < va.batch) {
                    member = next;
                    start_member();
                } else {
                    retired = true;
                }
            }
        }
        at_limit |= steps == va.max_steps;
        if (at_limit) {
            if (!kQueued) {
                if (__ballot(pc != kHalt)) my_error = PCVM_E_STEP_LIMIT;
                break;
            }
            if (pc != kHalt && steps - member_start >= va.max_steps) {  // this member does not halt: drop it
                my_error = PCVM_E_STEP_LIMIT;
                pc = kHalt;
                retired = true;
            }
        }
        int i;
        if (kQueued && va.policy == PCVM_SCHED_MOST_WAITING) {
            // largest count first, then the lowest block
            int best = 0;
            for (int b = 0; b < va.n_blocks; b += 8) {
                // (all eight comparisons first: a scalar instruction waits some 50 ticks for a mask that was just made)
                u64 at[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) at[u] = __builtin_amdgcn_uicmp((unsigned)pc, (unsigned)(b + u), 32);  // equal
                __builtin_amdgcn_sched_barrier(0);
                int k[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) k[u] = (__popcll(at[u]) << 8) + (kHalt - 1 - (b + u));
#pragma unroll
                for (int n = 4; n > 0; n /= 2)
#pragma unroll
                    for (int u = 0; u < n; ++u) k[u] = max(k[u], k[u + n]);
                best = max(best, k[0]);
            }
            i = best >= 256 ? kHalt - 1 - (best & 255) : kHalt;
        } else {
            i = wave_min(pc);
        }
        i = __builtin_amdgcn_readfirstlane(i);
        if (i == kHalt) break;
        const bool A = pc == i;  // locally active set
        const unsigned bx = __builtin_amdgcn_readlane(r_blkx, i), by = __builtin_amdgcn_readlane(r_blky, i);
        if (A) {
            bool failed = false;  // some lane is in error
            const int first = field(bx, 0, 255), end = first + field(bx, 8, 255);
            for (int k = first; k < end; ++k) {
                const unsigned ox = __builtin_amdgcn_readlane(r_opx, k), oy = __builtin_amdgcn_readlane(r_opy, k);
                const int kind = field(oy, 12, 15), ring_row = field(oy, 16, 255) * W;
                u64* const top = tops + field(oy, 0, 15) * kWave;
                unsigned* const count = counts + field(oy, 16, 255) * kWave;
                if (__builtin_expect(kind == PCVM_POP, 0)) {
                    const unsigned cnt = *count;
                    const int have = (int)(cnt & 0xffffu), low = (int)(cnt >> 16), idx = have - 2;  // entry that becomes the top
                    u64 x = rings[(ring_row + (idx & (W - 1))) * kWave];
                    unsigned n_cnt = cnt - 1;
                    if (__builtin_expect(__ballot(idx < low) != 0, 0)) {
                        if (idx < low) {  // below the ring, or no entry below the top
                            if (have >= 2) {
                                x = (u64)va.var_stacks[((size_t)field(oy, 16, 255) * va.depth + idx) * va.batch_pad + slot];
                                n_cnt = (unsigned)(have - 1) | ((unsigned)idx << 16);
                            } else {
                                x = *top;
                                if (have <= 0) {
                                    my_error = min(my_error, (int)PCVM_E_STACK_UNDERFLOW);
                                    n_cnt = cnt;
                                }
                            }
                        }
                        failed |= __ballot(my_error != 0) != 0;
                    }
                    *count = n_cnt;
                    *top = x;
                    continue;
                }
                const int cls = field(oy, 4, 15), push = kind == PCVM_PUSH ? 1 : 0;
                const u64 a = tops[ox & 0xffffu], b = rows[(ox >> 16) + (field(oy, 8, 1) ? 0 : lane)], old = *top;
                const unsigned cnt = *count;
                const u64 keep = cls == kClsMove ? 0ull : ~0ull, flip = cls == kClsSub ? ~0ull : 0ull;
                const u64 sum = (a & keep) + (b ^ flip) - flip;
                const bool lt = (long long)a < (long long)b, eq = a == b;
                const u64 rel = ((cls != kClsEq) & lt) | ((cls != kClsLt) & eq);
                u64 o = cls <= kClsSub ? sum : rel;
                if (__builtin_expect(cls > kClsEq, 0)) {
                    if (cls == kClsMul) {
                        o = a * b;
                    } else if (cls == kClsAnd) {
                        o = a & b;
                    } else if (cls == kClsShr) {
                        o = (u64)((long long)a >> (b & 63));
                    } else {
                        o = (b == 0 || b == ~0ull) ? 0ull : (u64)((long long)a % (long long)b);
                    }
                }
                const int have = (int)(cnt & 0xffffu), low = (int)(cnt >> 16), idx = have - 1;  // the old top goes below
                u64* e = push ? rings + (ring_row + (idx & (W - 1))) * kWave : rings - kWave;
                unsigned n_cnt = cnt + (unsigned)push;
                if (__builtin_expect(push && __ballot(have >= va.depth || idx - low >= W) != 0, 0)) {
                    if (have >= va.depth) {
                        my_error = min(my_error, (int)PCVM_E_STACK_OVERFLOW);
                        n_cnt = cnt;
                        o = old;
                        e = rings - kWave;
                    } else if (idx - low >= W) {  // the ring is full: its lowest entry makes room
                        va.var_stacks[((size_t)field(oy, 16, 255) * va.depth + (idx - W)) * va.batch_pad + slot] = (long long)*e;
                        n_cnt = (unsigned)(have + 1) | ((unsigned)(idx - W + 1) << 16);
                    }
                    failed |= __ballot(my_error != 0) != 0;
                }
                *e = old;  // (nobody reads it if there was no entry)
                *count = n_cnt;
                *top = o;
            }
            const int term = field(bx, 16, 15);
            if (__builtin_expect(term == PCVM_RETURN, 0)) {
                pc_sp -= 1;
                const int idx = pc_sp - 1;
                pc = pc_ring[(idx & (W - 1)) * kWave];
                if (__builtin_expect(__ballot(idx < pc_low) != 0, 0)) {
                    if (idx < pc_low) {
                        if (idx >= 0) {
                            pc = va.pc_stacks[(size_t)idx * va.batch_pad + slot];
                            pc_low = idx;
                        } else {
                            pc = kHalt;
                            if (kQueued && !my_error) va.outputs[member] = (long long)tops[va.output_var * kWave];
                        }
                    }
                }
            } else {
                const int call = term == PCVM_PUSHJUMP ? 1 : 0, idx = pc_sp - 1;
                const bool go_i = term != PCVM_BRANCH || tops[field(bx, 20, 15) * kWave] != 0;
                pc = go_i ? field(by, 0, 255) : field(by, 8, 255);
                int* e = call ? pc_ring + (idx & (W - 1)) * kWave : pc_ring - kWave;
                if (__builtin_expect(call && __ballot(pc_sp >= va.depth || idx - pc_low >= W) != 0, 0)) {
                    if (pc_sp >= va.depth) {
                        my_error = min(my_error, (int)PCVM_E_STACK_OVERFLOW);
                        e = pc_ring - kWave;
                    } else if (idx - pc_low >= W) {
                        va.pc_stacks[(size_t)(idx - W) * va.batch_pad + slot] = *e;
                        pc_low = idx - W + 1;
                    }
                    failed |= __ballot(my_error != 0) != 0;
                }
                *e = field(by, 8, 255);  // a call: where this frame resumes
                pc_sp += call;
            }
            if (__builtin_expect(failed, 0)) {  // a member in error stops; the others of its group go on
                if (my_error) {
                    pc = kHalt;
                    retired = true;
                }
            }
        }
        const int n_active = __popcll(__ballot(A));
        if (tracing && lane == 0 && steps < va.trace_capacity) {
            va.trace[2 * steps] = i;
            va.trace[2 * steps + 1] = n_active;
        }
        steps += 1;
        active_steps += (u64)n_active;
    }

    if (!kQueued && valid) va.outputs[member] = (long long)tops[va.output_var * kWave];
    if (my_error) atomicMin(va.error, my_error);
    if (lane == 0) {
        atomicAdd(&va.counters[0], (u64)steps);
        atomicAdd(&va.counters[1], active_steps);
    }
}

int check_program(const pcvm_program* p)
{
    if (!p || !p->blocks || (!p->ops && p->n_ops > 0)) return fail(PCVM_E_INVALID_ARG, "program, blocks and ops must not be NULL");
    if (p->n_vars < 1 || p->n_vars > PCVM_MAX_VARS) return fail(PCVM_E_INVALID_ARG, "n_vars must be in [1, %d]", PCVM_MAX_VARS);
    if (p->n_inputs < 1 || p->n_inputs > p->n_vars) return fail(PCVM_E_INVALID_ARG, "n_inputs must be in [1, n_vars]");
    if (p->output_var < 0 || p->output_var >= p->n_vars) return fail(PCVM_E_INVALID_ARG, "output_var out of range");
    if (p->n_blocks < 1 || p->n_blocks > (1 << 20)) return fail(PCVM_E_INVALID_ARG, "n_blocks out of range");
    if (p->n_ops < 0 || p->n_ops > (1 << 24)) return fail(PCVM_E_INVALID_ARG, "n_ops out of range");
    auto var_ok = [&](int v) { return v >= 0 && v < p->n_vars; };
    auto blk_ok = [&](int b) { return b >= 0 && b < p->n_blocks; };
    for (int b = 0; b < p->n_blocks; ++b) {
        const pcvm_block& k = p->blocks[b];
        if (k.first_op < 0 || k.n_ops < 0 || (long)k.first_op + k.n_ops > p->n_ops)
            return fail(PCVM_E_INVALID_ARG, "block %d: operations out of range", b);
        switch (k.term) {
        case PCVM_JUMP:
            if (!blk_ok(k.i)) return fail(PCVM_E_INVALID_ARG, "block %d: jump target out of range", b);
            break;
        case PCVM_BRANCH:
            if (!blk_ok(k.i) || !blk_ok(k.j) || !var_ok(k.x)) return fail(PCVM_E_INVALID_ARG, "block %d: bad branch", b);
            break;
        case PCVM_PUSHJUMP:
            if (!blk_ok(k.i) || !blk_ok(k.j)) return fail(PCVM_E_INVALID_ARG, "block %d: bad call", b);
            break;
        case PCVM_RETURN: break;
        default: return fail(PCVM_E_INVALID_ARG, "block %d: unknown terminator %d", b, k.term);
        }
    }
    for (int o = 0; o < p->n_ops; ++o) {
        const pcvm_op& op = p->ops[o];
        if (op.kind < PCVM_PUSH || op.kind > PCVM_POP) return fail(PCVM_E_INVALID_ARG, "operation %d: unknown kind %d", o, op.kind);
        if (!var_ok(op.dst)) return fail(PCVM_E_INVALID_ARG, "operation %d: destination out of range", o);
        if (op.kind == PCVM_POP) continue;
        if (op.fn < 0 || op.fn >= PCVM_FN_COUNT) return fail(PCVM_E_INVALID_ARG, "operation %d: unknown function %d", o, op.fn);
        if (!var_ok(op.a) || !var_ok(op.b)) return fail(PCVM_E_INVALID_ARG, "operation %d: operand out of range", o);
    }
    return PCVM_OK;
}

// Groups of a queued run of a small program, and the lanes of each that take members.  Up to one group per SIMD more
// groups cost nothing, and the fewer lanes share one the less they wait for each other (fibonacci, 3000 members: 1000 groups
// of 3 lanes 27.8 ms, 47 of 64 lanes 35.0).  Beyond that groups are full, three per SIMD: a step is latency, and so three
// hide behind each other (binomial, 176 408 members, EARLIEST: one group per SIMD 6.2 ms, three 4.7).
constexpr int kLdsBytes = 160 * 1024;
long queued_groups(long batch, int cus, int* lanes)
{
    const long simds = 4L * cus;
    *lanes = (int)std::min<long>(kWave, (batch + simds - 1) / simds);
    return std::min<long>(3 * simds, (batch + *lanes - 1) / *lanes);
}

// One device allocation per call, carved into the program tables, the stacks, the counters and the error word.
struct DeviceBuffers {
    void* base = nullptr;
    void* ptr[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    hipEvent_t ev[2] = {nullptr, nullptr};
    ~DeviceBuffers()
    {
        (void)hipFree(base);
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
    }
};

}  // namespace

extern "C" {

const char* pcvm_last_error(void) { return g_err; }

int pcvm_set_stream(void* hip_stream)
{
    g_stream = static_cast<hipStream_t>(hip_stream);
    return PCVM_OK;
}

static int run_impl(const pcvm_program* program, int64_t batch, const int64_t* inputs, int32_t stack_depth,
                    int64_t max_steps, int64_t* outputs, int32_t* trace, int64_t trace_capacity, pcvm_stats* stats,
                    bool queued, int policy)
{
    if (policy != PCVM_SCHED_EARLIEST && policy != PCVM_SCHED_MOST_WAITING) return fail(PCVM_E_INVALID_ARG, "unknown policy %d", policy);
    int rc = check_program(program);
    if (rc) return rc;
    if (batch < 1 || batch > (1ll << 28)) return fail(PCVM_E_INVALID_ARG, "batch must be in [1, 2^28]");
    if (!inputs || !outputs) return fail(PCVM_E_INVALID_ARG, "inputs and outputs must not be NULL");
    if (stack_depth < 1 || stack_depth > PCVM_MAX_DEPTH) return fail(PCVM_E_INVALID_ARG, "stack_depth must be in [1, %d]", PCVM_MAX_DEPTH);
    if (max_steps < 1) return fail(PCVM_E_INVALID_ARG, "max_steps must be > 0");
    if (trace && trace_capacity < 1) return fail(PCVM_E_INVALID_ARG, "trace_capacity must be > 0 with a trace buffer");
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count < 1)
        return fail(PCVM_E_DEVICE, "no HIP device available (this library has no CPU path)");

    long n_groups = (long)((batch + kWave - 1) / kWave);
    const bool small = small_program(program);
    SmallTables tables;
    SmallArgs sm{};
    size_t small_lds = 0;
    if (small) {
        int cus = 0, dev = 0;
        PCVM_TRY(hipGetDevice(&dev), PCVM_E_DEVICE);
        PCVM_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), PCVM_E_DEVICE);
        sm.n_stacks = pack_small(program, &tables);
        sm.lanes = kWave;
        if (queued) n_groups = queued_groups(batch, cus, &sm.lanes);
        // as long a ring as the workgroups of a compute unit can share its LDS for (up to four of them: the registers
        // allow no more to be useful)
        const long wgs = (n_groups + kWavesPerBlock - 1) / kWavesPerBlock;
        const long share = std::min<long>(4, (wgs + cus - 1) / cus);
        auto lds = [&](int ring) { return kWavesPerBlock * small_wave_bytes(program->n_vars, sm.n_stacks, ring); };
        sm.ring = 1;
        while (sm.ring < stack_depth && lds(2 * sm.ring) <= (size_t)(kLdsBytes / share)) sm.ring *= 2;
        small_lds = lds(sm.ring);
        const void* fn = queued ? reinterpret_cast<const void*>(pcvm_small_kernel<true>) : reinterpret_cast<const void*>(pcvm_small_kernel<false>);
        PCVM_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes), PCVM_E_DEVICE);
    } else if (queued) {  // no more groups than the chip holds at once: the others' members come through the queue
        int per_cu = 0, cus = 0, dev = 0;
        PCVM_TRY(hipGetDevice(&dev), PCVM_E_DEVICE);
        PCVM_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, pcvm_kernel<true>, kWave * kWavesPerBlock, 0), PCVM_E_DEVICE);
        PCVM_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), PCVM_E_DEVICE);
        const long resident = (long)(per_cu < 1 ? 1 : per_cu) * cus * kWavesPerBlock;
        if (n_groups > resident) n_groups = resident;
    }
    const long batch_pad = n_groups * (small && queued ? sm.lanes : kWave);
    // (a small program keeps stacks of the variables that are pushed only, and none in memory where the rings hold them all)
    const bool deep = !small || sm.ring < stack_depth;
    const size_t var_bytes = deep ? (size_t)(small ? sm.n_stacks : program->n_vars) * stack_depth * batch_pad * sizeof(long long) : 0;
    const size_t pc_bytes = deep ? (size_t)stack_depth * batch_pad * sizeof(int) : 0;
    // (what is refused does not depend on how little of it a program really takes)
    const size_t lanes = (size_t)std::min<long>(n_groups * kWave, (long)((batch + kWave - 1) / kWave * kWave));
    const size_t most = ((size_t)program->n_vars * sizeof(long long) + sizeof(int)) * stack_depth * lanes;
    if (most > (size_t)64 << 30) return fail(PCVM_E_ALLOC, "stacks would need %zu bytes", most);

    DeviceBuffers buf;
    {
        const size_t part[6] = {small ? sizeof(SmallTables) : sizeof(pcvm_block) * program->n_blocks, sizeof(pcvm_op) * (program->n_ops > 0 ? program->n_ops : 1),
                                var_bytes, pc_bytes, 3 * sizeof(unsigned long long), sizeof(int)};
        size_t off[6], total = 0;
        for (int i = 0; i < 6; ++i) {
            off[i] = total;
            total += (part[i] + 255) & ~(size_t)255;
        }
        PCVM_TRY(hipMalloc(&buf.base, total), PCVM_E_ALLOC);
        for (int i = 0; i < 6; ++i) buf.ptr[i] = static_cast<char*>(buf.base) + off[i];
    }
    PCVM_TRY(hipEventCreate(&buf.ev[0]), PCVM_E_DEVICE);
    PCVM_TRY(hipEventCreate(&buf.ev[1]), PCVM_E_DEVICE);
    if (small)
        PCVM_TRY(hipMemcpyAsync(buf.ptr[0], &tables, sizeof(SmallTables), hipMemcpyHostToDevice, g_stream), PCVM_E_DEVICE);
    else
        PCVM_TRY(hipMemcpyAsync(buf.ptr[0], program->blocks, sizeof(pcvm_block) * program->n_blocks, hipMemcpyHostToDevice, g_stream), PCVM_E_DEVICE);
    if (!small && program->n_ops > 0)
        PCVM_TRY(hipMemcpyAsync(buf.ptr[1], program->ops, sizeof(pcvm_op) * program->n_ops, hipMemcpyHostToDevice, g_stream), PCVM_E_DEVICE);
    PCVM_TRY(hipMemsetAsync(buf.ptr[4], 0, 3 * sizeof(unsigned long long), g_stream), PCVM_E_DEVICE);
    PCVM_TRY(hipMemsetAsync(buf.ptr[5], 0, sizeof(int), g_stream), PCVM_E_DEVICE);

    VmArgs va{};
    va.blocks = static_cast<const pcvm_block*>(buf.ptr[0]);
    va.ops = static_cast<const pcvm_op*>(buf.ptr[1]);
    va.n_vars = program->n_vars;
    va.n_inputs = program->n_inputs;
    va.output_var = program->output_var;
    va.n_blocks = program->n_blocks;
    va.batch = (long)batch;
    va.batch_pad = batch_pad;
    va.depth = stack_depth;
    va.max_steps = (long)max_steps;
    va.inputs = reinterpret_cast<const long long*>(inputs);
    va.outputs = reinterpret_cast<long long*>(outputs);
    va.var_stacks = static_cast<long long*>(buf.ptr[2]);
    va.pc_stacks = static_cast<int*>(buf.ptr[3]);
    va.trace = trace;
    va.trace_capacity = (long)trace_capacity;
    va.counters = static_cast<unsigned long long*>(buf.ptr[4]);
    va.queue = va.counters + 2;
    va.policy = policy;
    va.error = static_cast<int*>(buf.ptr[5]);

    const unsigned blocks = (unsigned)((n_groups + kWavesPerBlock - 1) / kWavesPerBlock);
    PCVM_TRY(hipEventRecord(buf.ev[0], g_stream), PCVM_E_DEVICE);
    sm.tables = static_cast<const SmallTables*>(buf.ptr[0]);
    if (small && queued)
        hipLaunchKernelGGL(pcvm_small_kernel<true>, dim3(blocks), dim3(kWave * kWavesPerBlock), small_lds, g_stream, va, sm);
    else if (small)
        hipLaunchKernelGGL(pcvm_small_kernel<false>, dim3(blocks), dim3(kWave * kWavesPerBlock), small_lds, g_stream, va, sm);
    else if (queued)
        hipLaunchKernelGGL(pcvm_kernel<true>, dim3(blocks), dim3(kWave * kWavesPerBlock), 0, g_stream, va);
    else
        hipLaunchKernelGGL(pcvm_kernel<false>, dim3(blocks), dim3(kWave * kWavesPerBlock), 0, g_stream, va);
    PCVM_TRY(hipGetLastError(), PCVM_E_DEVICE);
    PCVM_TRY(hipEventRecord(buf.ev[1], g_stream), PCVM_E_DEVICE);
    unsigned long long counters[2] = {0, 0};
    int error = 0;
    PCVM_TRY(hipMemcpyAsync(counters, buf.ptr[4], sizeof(counters), hipMemcpyDeviceToHost, g_stream), PCVM_E_DEVICE);
    PCVM_TRY(hipMemcpyAsync(&error, buf.ptr[5], sizeof(error), hipMemcpyDeviceToHost, g_stream), PCVM_E_DEVICE);
    PCVM_TRY(hipStreamSynchronize(g_stream), PCVM_E_DEVICE);
    if (stats) {
        float ms = 0.f;
        PCVM_TRY(hipEventElapsedTime(&ms, buf.ev[0], buf.ev[1]), PCVM_E_DEVICE);
        stats->steps = counters[0];
        stats->active_member_steps = counters[1];
        stats->issued_member_steps = counters[0] * kWave;
        stats->kernel_ms = ms;
        stats->n_groups = (int32_t)n_groups;
        stats->reserved = 0;
    }
    if (error == PCVM_E_STACK_OVERFLOW) return fail(error, "a stack grew beyond stack_depth = %d entries", stack_depth);
    if (error == PCVM_E_STACK_UNDERFLOW) return fail(error, "pop from an empty variable stack");
    if (error == PCVM_E_STEP_LIMIT) return fail(error, "a group made %lld steps without halting", (long long)max_steps);
    if (error) return fail(PCVM_E_DEVICE, "unknown device error %d", error);
    return PCVM_OK;
}

int pcvm_run(const pcvm_program* program, int64_t batch, const int64_t* inputs, int32_t stack_depth,
             int64_t max_steps, int64_t* outputs, int32_t* trace, int64_t trace_capacity, pcvm_stats* stats)
{
    return run_impl(program, batch, inputs, stack_depth, max_steps, outputs, trace, trace_capacity, stats, false,
                    PCVM_SCHED_EARLIEST);
}

int pcvm_run_queued(const pcvm_program* program, int64_t batch, const int64_t* inputs, int32_t stack_depth,
                    int64_t max_steps, int32_t policy, int64_t* outputs, pcvm_stats* stats)
{
    return run_impl(program, batch, inputs, stack_depth, max_steps, outputs, nullptr, 0, stats, true, policy);
}

}  // extern "C"
