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
// Programs of up to 64 blocks and 64 operations take pcvm_small_kernel, which keeps all of that in registers and LDS and runs
// its steps in a piece of assembly.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <type_traits>
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

// ---- programs whose records fit the lanes of a wave ----
//
// A step is a serial chain - choose a block, fetch its record, run its operations one after the other, go on - and a
// batch lasts as long as its longest member.  A wave issues an instruction every five ticks at best, vector or scalar alike,
// and waits for the instruction memory at every branch that is taken, so what bounds a step is how many instructions and
// branches the interpreter spends on it (fibonacci: 280 instructions, 1900 ticks a block, as the compiler laid out an
// interpreter with its tops in LDS; 165, 1220 with the tops in registers).  So
//   * steps run in one piece of assembly that is left only for what is rare: stacks that need memory, errors, members
//     that halt, the step limit (StepLoop below),
//   * an operation, a call and the end of a block are entries of one table, lane k of a few registers holding entry k (and of
//     a second set of them entry 64 + k, where a program has more), and an entry names the handler that runs it: one jump an entry, to code that knows what it is,
//   * the tops and the counts of the stacks are in registers, which the entry's word picks through the register index
//     mode as it stands (s_set_gpr_idx_on takes the low eight bits of a scalar): no field to extract, no address, no wait,
//   * the entries below a top are in a ring of `ring` entries per stack in LDS, and the return addresses, of as many bits as
//     the program's blocks need, in a pair of registers; only what a deeper push drives out goes to global memory, and only a pop that reaches below
//     the ring reads it back.  One comparison per push or pop finds both that and every error,
//   * the block most lanes wait for is found by counting lanes block by block; under that policy a block that is entered
//     by a jump or a call runs together with the one before it (the lanes that arrive there are as many as had just been the
//     most), so that a call of fibonacci takes four choices instead of six.
// A block of fibonacci is 88 instructions and 680 ticks so.  200 000 members, queued, MOST_WAITING: fibonacci 37.2 -> 17.9 ms,
// collatz_steps 0.98 -> 0.30, gcd 0.75 -> 0.36, binomial 3.96 -> 1.47; 3000 members 27.9 -> 10.0, 0.61 -> 0.18, 0.112 -> 0.058,
// 1.85 -> 0.71; 200 000 in fixed groups 33.2 -> 17.9, 0.73 -> 0.34, 0.193 -> 0.196 (deep stacks, through memory), 4.1 -> 2.3.
constexpr int kSmallMax = 64;       // blocks
constexpr int kEntries = 2 * kSmallMax;  // as many as 64 operations and the ends of 64 blocks take

// Blocks are named by codes, block b by 63 - b, so that the lowest block has the largest code; a lane that waits for none
// (the counting below asks for a code of -1 and of -2 too, where there are 64 blocks: no lane may have them):
constexpr int kHalt = -16, kRetired = -17;  // its member has halted; in queued runs, there is none left for it
constexpr int code_of(int block) { return kSmallMax - 1 - block; }

// An entry: word = {operand a or variable | destination << 8 | handler << 24}, two immediates (the 64-bit immediate, or
// operand b in the first; of a branch the codes of i and j; of a jump its target's; of a call the resuming block, and
// of one that ends a record its target's), and the stack it works on.  Handlers: a value's kind, plus 16 where the value is pushed; and
enum : int { kValConst = 0, kValAddImm, kValLeImm, kValEqImm, kValAdd, kValSub, kValLe, kValLt, kValEq, kValMul, kValMulImm, kValAndImm, kValShrImm, kValMod };
enum : int { kDoPop = 14, kDoCall = 15, kDoPush = 16, kDoJump = 30, kDoBranch = 31, kDoReturn = 32, kDoCallJump = 33 };
struct SmallTables {
    unsigned input_stacks;  // bit v: variable v has a stack and is an input
    // record: {first entry | blocks that it runs << 8}, of block b in lane 63 - b; stack: of entry k in lane k + 1
    unsigned word[kEntries], imm_lo[kEntries], imm_hi[kEntries], stack[kEntries], record[kSmallMax];
    int n_entries;
};

int value_kind(int fn)
{
    switch (fn) {
    case PCVM_CONST: return kValConst;
    case PCVM_COPY: return kValAddImm;  // (its immediate is packed as 0)
    case PCVM_ADD: return kValAdd;
    case PCVM_SUB: return kValSub;
    case PCVM_MUL: return kValMul;
    case PCVM_ADDI: return kValAddImm;
    case PCVM_MULI: return kValMulImm;
    case PCVM_LE: return kValLe;
    case PCVM_LT: return kValLt;
    case PCVM_EQ: return kValEq;
    case PCVM_LEI: return kValLeImm;
    case PCVM_EQI: return kValEqImm;
    case PCVM_MOD: return kValMod;
    case PCVM_ANDI: return kValAndImm;
    default: return kValShrImm;  // PCVM_SHRI
    }
}

// Blocks that run together with block b: itself and, if `join`, those that the end before them enters unconditionally.
// No more operations than stack_depth, and one call at the most: a push that fails cannot be followed by as many pops, so
// that an error is the one of the block it happens in.
std::vector<int> joined_blocks(const pcvm_program* p, int b, bool join, int stack_depth)
{
    std::vector<int> chain{b};
    bool called = false;
    int n_ops = p->blocks[b].n_ops;
    while (join && chain.size() < 4) {
        const pcvm_block& k = p->blocks[chain.back()];
        if (k.term != PCVM_JUMP && k.term != PCVM_PUSHJUMP) break;
        const pcvm_block& t = p->blocks[k.i];
        called |= k.term == PCVM_PUSHJUMP;
        if (called && t.term == PCVM_PUSHJUMP) break;
        if (std::find(chain.begin(), chain.end(), k.i) != chain.end() || n_ops + t.n_ops > stack_depth) break;
        n_ops += t.n_ops;
        chain.push_back(k.i);
    }
    return chain;
}

// Returns the number of variables that keep a stack (those that are pushed or popped), or -1 if the program has more blocks
// than there are lanes, or more entries than fit.  (Joined blocks are given up before the second set of registers is used.)
int pack_small(const pcvm_program* p, bool join, int stack_depth, SmallTables* t)
{
    *t = SmallTables{};
    if (p->n_blocks > kSmallMax) return -1;
    int stack_of[PCVM_MAX_VARS], n_stacks = 0, n = 0;
    for (int v = 0; v < PCVM_MAX_VARS; ++v) stack_of[v] = -1;
    for (int o = 0; o < p->n_ops; ++o)
        if (p->ops[o].kind != PCVM_UPDATE && stack_of[p->ops[o].dst] < 0) stack_of[p->ops[o].dst] = n_stacks++;
    for (int v = 0; v < p->n_inputs; ++v)
        if (stack_of[v] >= 0) t->input_stacks |= 1u << v;
    auto entry = [&](int handler, int a, int dst, unsigned long long imm, int stack) {
        if (n < kEntries) {
            t->word[n] = (unsigned)a | (unsigned)dst << 8 | (unsigned)handler << 24;
            t->imm_lo[n] = (unsigned)imm;
            t->imm_hi[n] = (unsigned)(imm >> 32);
            t->stack[(n + 1) % kEntries] = (unsigned)(stack < 0 ? 0 : stack);
        }
        ++n;
    };
    for (int b = 0; b < p->n_blocks && n <= kEntries; ++b) {
        const std::vector<int> chain = joined_blocks(p, b, join, stack_depth);
        t->record[code_of(b)] = (unsigned)n | (unsigned)chain.size() << 8;
        for (int c : chain) {
            const pcvm_block& k = p->blocks[c];
            for (int o = k.first_op; o < k.first_op + k.n_ops && n <= kEntries; ++o) {
                const pcvm_op& op = p->ops[o];
                if (op.kind == PCVM_POP) {
                    entry(kDoPop, 0, op.dst, 0, stack_of[op.dst]);
                    continue;
                }
                const int kind = value_kind(op.fn);
                const bool two = kind == kValMod || kind == kValMul || (kind >= kValAdd && kind <= kValEq);
                const unsigned long long imm = two ? (unsigned long long)op.b : op.fn == PCVM_COPY ? 0ull : (unsigned long long)op.imm;
                entry(kind + (op.kind == PCVM_PUSH ? kDoPush : 0), op.a, op.dst, imm, stack_of[op.dst]);
            }
            if (k.term == PCVM_PUSHJUMP && c != chain.back()) entry(kDoCall, 0, 0, (unsigned)k.j, -1);
        }
        const pcvm_block& end = p->blocks[chain.back()];
        if (end.term == PCVM_BRANCH)
            entry(kDoBranch, end.x, 0, (unsigned)code_of(end.i) | (unsigned long long)(unsigned)code_of(end.j) << 32, -1);
        else if (end.term == PCVM_RETURN)
            entry(kDoReturn, 0, 0, 0, -1);
        else if (end.term == PCVM_PUSHJUMP)
            entry(kDoCallJump, 0, 0, (unsigned)end.j | (unsigned long long)(unsigned)code_of(end.i) << 32, -1);
        else
            entry(kDoJump, 0, 0, (unsigned)code_of(end.i), -1);
    }
    t->n_entries = n;
    if (n <= (join ? kSmallMax : kEntries)) return n_stacks;
    return join ? pack_small(p, false, stack_depth, t) : -1;
}

struct SmallArgs {
    const SmallTables* tables;
    int n_stacks;
    int ring;   // entries per stack in LDS, a power of two
    int lanes;  // queued runs: lanes of a group that take members
    int frame_bits, frames;  // bits of a return address, and how many of them two registers hold
};

// LDS of a wave: rings [stack][entry][lane].
__host__ __device__ inline size_t small_wave_bytes(int n_stacks, int ring)
{
    return (size_t)(n_stacks > 0 ? n_stacks : 1) * 8 * ring * kWave;
}

// The register files: tops (low words in v68 and on, high words in v84 and on) and counts (v100 and on) of the variables'
// stacks, {entries | index of the lowest one that is in the ring << 16}; v116 to v127 are the handlers' own.  They are
// registers that the compiler does not know of: only by its number can a register be the base of an access in the register
// index mode.  The limit of 64 registers that eight waves per SIMD stand for keeps the compiler below them (with four to spare,
// for the registers in which it parks scalars come on top of its limit), and the clobber of the last one makes the kernel own
// them: four waves per SIMD.  `w` picks the variable with its low eight bits (the index mode keeps them in M0).
__device__ __forceinline__ void file_own() { asm volatile("" ::: "v127"); }
__device__ __forceinline__ unsigned long long file_read(unsigned w, unsigned& c)
{
    unsigned l, h;
    asm volatile("s_set_gpr_idx_on %3, gpr_idx(SRC0)\n\tv_mov_b32 %0, v68\n\tv_mov_b32 %1, v84\n\tv_mov_b32 %2, v100\n\ts_set_gpr_idx_off"
                 : "=&v"(l), "=&v"(h), "=&v"(c)
                 : "s"(w)
                 : "m0");
    return (unsigned long long)l | (unsigned long long)h << 32;
}
__device__ __forceinline__ unsigned long long file_read(unsigned w)
{
    unsigned c;
    return file_read(w, c);
}
__device__ __forceinline__ void file_write(unsigned w, unsigned long long x, unsigned c)
{
    asm volatile("s_set_gpr_idx_on %3, gpr_idx(DST)\n\tv_mov_b32 v68, %0\n\tv_mov_b32 v84, %1\n\tv_mov_b32 v100, %2\n\ts_set_gpr_idx_off" ::"v"((unsigned)x),
                 "v"((unsigned)(x >> 32)), "v"(c), "s"(w)
                 : "m0");
}

// ---- the step loop ----
// Scalars: s[40:41] handlers, s[42:43] the handler to go to, s[44:45] immediates, s46 the entry's word, s47 the next one's,
// s48 its destination, s49 its ring's rows; s50 and on: choosing.  Vectors: v[116:117] value, v[118:119] operand b or the
// old top, v120 count, v121 address,
// v[122:127] the remainder's.  The instructions between a vector one that writes a scalar and a vector one that reads
// it (two, or four for a lane select) are counted by hand here: the compiler looks into no assembly.
// (handler h is 512 h bytes behind handler 0; the assembler refuses one that is longer)
#define VM_AT(h) ".org vm_h0_%=+" #h "*512\n"
// (B fetches the next entry's word while this one runs, N goes there, R fetches the rows of this one's stack; with entries
// in two sets of registers bit 6 of the index says which)
#define VM_GO "s_lshr_b32 s42, s47, 15\ns_add_u32 s42, s40, s42\ns_addc_u32 s43, s41, 0\n"
#define VM_GONE "s_add_u32 %[k], %[k], 1\ns_mov_b32 s46, s47\ns_setpc_b64 s[42:43]\n"
#define VM_B1 "v_readlane_b32 s47, %[word], %[k]\n"
#define VM_N1 VM_GO "v_readlane_b32 s44, %[lo], %[k]\nv_readlane_b32 s45, %[hi], %[k]\n" VM_GONE
#define VM_R1 "v_readlane_b32 s49, %[row], %[k]\n"
#define VM_EITHER(s, name) "v_readlane_b32 " s ", %[" name "], %[k]\nv_readlane_b32 s51, %[" name "2], %[k]\ns_bitcmp1_b32 %[k], 6\ns_cselect_b32 " s ", s51, " s "\n"
#define VM_B2 VM_EITHER("s47", "word")
#define VM_N2 "s_branch vm_next_%=\n"
#define VM_T2 "vm_next_%=:\n" VM_GO VM_EITHER("s44", "lo") VM_EITHER("s45", "hi") VM_GONE
#define VM_R2 VM_EITHER("s49", "row")
#define VM_DONE "s_mov_b64 exec, -1\ns_branch vm_head_%=\n"
#define VM_RARE "s_cbranch_vccnz vm_rare_%=\n"
#define VM_A "s_set_gpr_idx_on s46, gpr_idx(SRC0)\nv_mov_b32 v116, v68\nv_mov_b32 v117, v84\ns_set_gpr_idx_off\n"
#define VM_AB VM_A "s_set_gpr_idx_on s44, gpr_idx(SRC0)\nv_mov_b32 v118, v68\nv_mov_b32 v119, v84\ns_set_gpr_idx_off\n"
#define VM_BOOL "v_mov_b32 v117, 0\ns_nop 0\nv_cndmask_b32_e64 v116, 0, 1, vcc\n"
#define VM_CONST "v_mov_b32 v116, s44\nv_mov_b32 v117, s45\n"
#define VM_ADDI VM_A "v_lshl_add_u64 v[116:117], v[116:117], 0, s[44:45]\n"
#define VM_LEI VM_A "v_cmp_ge_i64 vcc, s[44:45], v[116:117]\n" VM_BOOL
#define VM_EQI VM_A "v_cmp_eq_u64 vcc, s[44:45], v[116:117]\n" VM_BOOL
#define VM_ADD VM_AB "v_lshl_add_u64 v[116:117], v[116:117], 0, v[118:119]\n"
#define VM_SUB VM_AB "v_sub_co_u32 v116, vcc, v116, v118\ns_nop 1\nv_subb_co_u32 v117, vcc, v117, v119, vcc\n"
#define VM_LE VM_AB "v_cmp_le_i64 vcc, v[116:117], v[118:119]\n" VM_BOOL
#define VM_LT VM_AB "v_cmp_lt_i64 vcc, v[116:117], v[118:119]\n" VM_BOOL
#define VM_EQ VM_AB "v_cmp_eq_u64 vcc, v[116:117], v[118:119]\n" VM_BOOL
#define VM_TIMES                                                                                                            \
    "v_mul_lo_u32 v121, v116, v119\nv_mul_lo_u32 v117, v117, v118\nv_add_u32 v121, v121, v117\n"                            \
    "v_mul_hi_u32 v117, v116, v118\nv_mul_lo_u32 v116, v116, v118\nv_add_u32 v117, v117, v121\n"
#define VM_MUL VM_AB VM_TIMES
#define VM_MULI VM_A "v_mov_b32 v118, s44\nv_mov_b32 v119, s45\n" VM_TIMES
#define VM_ANDI VM_A "v_and_b32 v116, s44, v116\nv_and_b32 v117, s45, v117\n"
#define VM_SHRI VM_A "v_ashrrev_i64 v[116:117], s44, v[116:117]\n"
// (of two numbers below 2^32, by the reciprocal of the divisor in binary64: the quotient less a half, rounded down, is right
// or one too small.  Larger or negative ones, and a divisor of 0, are left to the compiler's division.)
#define VM_MOD                                                                                                              \
    "v_or_b32 v121, v117, v119\nv_cmp_ne_u32 vcc, 0, v121\ns_cbranch_vccnz vm_modulo_%=\nv_cmp_eq_u32 vcc, 0, v118\n"       \
    "s_cbranch_vccnz vm_modulo_%=\nv_cvt_f64_u32 v[120:121], v116\nv_cvt_f64_u32 v[122:123], v118\n"                       \
    "v_rcp_f64 v[124:125], v[122:123]\ns_nop 1\nv_fma_f64 v[126:127], -v[122:123], v[124:125], 1.0\n"                      \
    "v_fma_f64 v[124:125], v[126:127], v[124:125], v[124:125]\nv_fma_f64 v[126:127], -v[122:123], v[124:125], 1.0\n"       \
    "v_fma_f64 v[124:125], v[126:127], v[124:125], v[124:125]\nv_fma_f64 v[120:121], v[120:121], v[124:125], -0.5\n"       \
    "v_cvt_u32_f64 v120, v[120:121]\nv_mul_lo_u32 v120, v120, v118\nv_sub_u32 v116, v116, v120\n"                          \
    "v_sub_u32 v120, v116, v118\nv_min_u32 v116, v116, v120\n"
#define VM_UPDATE "s_lshr_b32 s48, s46, 8\ns_set_gpr_idx_on s48, gpr_idx(DST)\nv_mov_b32 v68, v116\nv_mov_b32 v84, v117\ns_set_gpr_idx_off\n"
#define VM_SET_ALL "s_set_gpr_idx_on s48, gpr_idx(DST)\nv_mov_b32 v68, v116\nv_mov_b32 v84, v117\nv_mov_b32 v100, v120\ns_set_gpr_idx_off\n"
// (address of ring entry v121, entries counted modulo the ring)
#define VM_SLOT "v_and_b32 v121, %[mask], v121\nv_lshl_add_u32 v121, v121, 9, %[base]\nv_add_u32 v121, s49, v121\n"
#define VM_IN_RING "v_sub_u32_sdwa v121, v120, v120 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1\n"
#define VM_PUSH(R)                                                                                                             \
    R "s_lshr_b32 s48, s46, 8\ns_set_gpr_idx_on s48, gpr_idx(SRC0)\nv_mov_b32 v120, v100\n"  \
    "v_mov_b32 v118, v68\nv_mov_b32 v119, v84\ns_set_gpr_idx_off\n" VM_IN_RING "v_cmp_le_i32 vcc, %[full], v121\n" VM_RARE  \
    "v_add_u32 v121, -1, v120\n" VM_SLOT "ds_write_b64 v121, v[118:119]\nv_add_u32 v120, 1, v120\n" VM_SET_ALL
#define VM_POP(R)                                                                                                              \
    R "s_lshr_b32 s48, s46, 8\ns_set_gpr_idx_on s48, gpr_idx(SRC0)\nv_mov_b32 v120, v100\n"  \
    "s_set_gpr_idx_off\n" VM_IN_RING "v_cmp_ge_i32 vcc, 1, v121\n" VM_RARE "v_add_u32 v121, -2, v120\n" VM_SLOT             \
    "ds_read_b64 v[116:117], v121\nv_add_u32 v120, -1, v120\ns_waitcnt lgkmcnt(0)\n" VM_SET_ALL
#define VM_CALL                                                                                                             \
    "v_alignbit_b32 %[f_hi], %[f_hi], %[f_lo], %[f_up]\nv_lshlrev_b32 %[f_lo], %[f_down], %[f_lo]\n"                        \
    "v_or_b32 %[f_lo], s44, %[f_lo]\nv_add_u32 %[held], 1, %[held]\n"
#define VM_HANDLERS(B, N, R)                                                                                                         \
    ".p2align 8\nvm_h0_%=:\n" B VM_CONST VM_UPDATE N VM_AT(1) B VM_ADDI VM_UPDATE N                                \
    VM_AT(2) B VM_LEI VM_UPDATE N VM_AT(3) B VM_EQI VM_UPDATE N                                   \
    VM_AT(4) B VM_ADD VM_UPDATE N VM_AT(5) B VM_SUB VM_UPDATE N                                   \
    VM_AT(6) B VM_LE VM_UPDATE N VM_AT(7) B VM_LT VM_UPDATE N                                     \
    VM_AT(8) B VM_EQ VM_UPDATE N VM_AT(9) B VM_MUL VM_UPDATE N                                    \
    VM_AT(10) B VM_MULI VM_UPDATE N VM_AT(11) B VM_ANDI VM_UPDATE N                               \
    VM_AT(12) B VM_SHRI VM_UPDATE N VM_AT(13) B VM_AB VM_MOD "vm_update_%=:\n" VM_UPDATE N                                        \
    VM_AT(14) B VM_POP(R) N                                                                                       \
    VM_AT(15) B "v_cmp_ge_i32 vcc, %[held], %[held_max]\n" VM_RARE                                                  \
    VM_CALL N                                              \
    VM_AT(16) B VM_CONST VM_PUSH(R) N VM_AT(17) B VM_ADDI VM_PUSH(R) N                                  \
    VM_AT(18) B VM_LEI VM_PUSH(R) N VM_AT(19) B VM_EQI VM_PUSH(R) N                                     \
    VM_AT(20) B VM_ADD VM_PUSH(R) N VM_AT(21) B VM_SUB VM_PUSH(R) N                                     \
    VM_AT(22) B VM_LE VM_PUSH(R) N VM_AT(23) B VM_LT VM_PUSH(R) N                                       \
    VM_AT(24) B VM_EQ VM_PUSH(R) N VM_AT(25) B VM_MUL VM_PUSH(R) N VM_AT(26) B VM_MULI VM_PUSH(R) N             \
    VM_AT(27) B VM_ANDI VM_PUSH(R) N VM_AT(28) B VM_SHRI VM_PUSH(R) N VM_AT(29) B VM_AB VM_MOD "vm_push_%=:\n" VM_PUSH(R) N \
    VM_AT(30) "v_mov_b32 %[pc], s44\n" VM_DONE                                                                              \
    VM_AT(31) VM_A "v_or_b32 v116, v116, v117\nv_mov_b32 v118, s44\nv_mov_b32 v119, s45\nv_cmp_ne_u32 vcc, 0, v116\n"       \
    "s_nop 1\nv_cndmask_b32 %[pc], v119, v118, vcc\n" VM_DONE                                                               \
    VM_AT(32) "v_cmp_ge_i32 vcc, 0, %[held]\n" VM_RARE                                                                       \
    "v_and_b32 v116, %[f_mask], %[f_lo]\nv_alignbit_b32 %[f_lo], %[f_hi], %[f_lo], %[f_down]\nv_add_u32 %[held], -1, %[held]\n" \
    "v_lshrrev_b32 %[f_hi], %[f_down], %[f_hi]\nv_sub_u32 %[pc], 63, v116\n" VM_DONE                                                                          \
    VM_AT(33) "v_cmp_ge_i32 vcc, %[held], %[held_max]\n" VM_RARE VM_CALL "v_mov_b32 %[pc], s45\n" VM_DONE

// Choosing: s50 = {lanes that wait | code} of the block most of them wait for, the largest code on a tie ...
#define VM_COUNT(s, c) "v_cmp_eq_u32 s[" s "], " c ", %[pc]\n"
#define VM_CHOOSE_MOST                                                                                                      \
    VM_COUNT("52:53", "63") VM_COUNT("54:55", "62") VM_COUNT("56:57", "61") VM_COUNT("58:59", "60") VM_COUNT("60:61", "59") \
    VM_COUNT("62:63", "58")                                                                                                 \
    "s_bcnt1_i32_b64 s52, s[52:53]\ns_bcnt1_i32_b64 s54, s[54:55]\ns_bcnt1_i32_b64 s56, s[56:57]\n"                         \
    "s_bcnt1_i32_b64 s58, s[58:59]\ns_bcnt1_i32_b64 s60, s[60:61]\ns_bcnt1_i32_b64 s62, s[62:63]\n"                         \
    "s_pack_ll_b32_b16 s52, 63, s52\ns_pack_ll_b32_b16 s54, 62, s54\ns_pack_ll_b32_b16 s56, 61, s56\n"                      \
    "s_pack_ll_b32_b16 s58, 60, s58\ns_pack_ll_b32_b16 s60, 59, s60\ns_pack_ll_b32_b16 s62, 58, s62\n"                      \
    "s_max_u32 s52, s52, s54\ns_max_u32 s56, s56, s58\ns_max_u32 s60, s60, s62\ns_max_u32 s52, s52, s56\n"                  \
    "s_max_u32 s50, s52, s60\ns_cmp_gt_i32 %[lowest], 57\ns_cbranch_scc1 vm_chosen_%=\ns_mov_b32 s60, 57\n"                 \
    "vm_count_%=:\n"                                                                                                        \
    "s_add_i32 s61, s60, -1\ns_add_i32 s62, s60, -2\n" VM_COUNT("52:53", "s60") VM_COUNT("54:55", "s61")                    \
    VM_COUNT("56:57", "s62")                                                                                                \
    "s_bcnt1_i32_b64 s52, s[52:53]\ns_bcnt1_i32_b64 s54, s[54:55]\ns_bcnt1_i32_b64 s56, s[56:57]\n"                         \
    "s_pack_ll_b32_b16 s52, s60, s52\ns_pack_ll_b32_b16 s54, s61, s54\ns_pack_ll_b32_b16 s56, s62, s56\n"                   \
    "s_max_u32 s52, s52, s54\ns_max_u32 s50, s50, s56\ns_add_i32 s60, s60, -3\ns_max_u32 s50, s50, s52\n"                   \
    "s_cmp_ge_i32 s60, %[lowest]\ns_cbranch_scc1 vm_count_%=\n"                                                             \
    "vm_chosen_%=:\n"
#define VM_NONE_MOST "s_cmp_lt_u32 s50, 0x10000\ns_cbranch_scc1 vm_none_%=\n"
// ... or the earliest block that any lane waits for: its code is the largest.
#define VM_ROW_MAX(n) "s_nop 1\nv_max_i32_dpp v116, v116, v116 row_ror:" n " row_mask:0xf bank_mask:0xf\n"
#define VM_CHOOSE_EARLIEST                                                                                                  \
    "v_mov_b32 v116, %[pc]\n" VM_ROW_MAX("8") VM_ROW_MAX("4") VM_ROW_MAX("2") VM_ROW_MAX("1")                               \
    "s_nop 1\nv_readlane_b32 s50, v116, 0\nv_readlane_b32 s51, v116, 16\nv_readlane_b32 s52, v116, 32\n"                    \
    "v_readlane_b32 s53, v116, 48\ns_max_i32 s50, s50, s51\ns_max_i32 s52, s52, s53\ns_max_i32 s50, s50, s52\n"
#define VM_NONE_EARLIEST "s_cmp_lt_i32 s50, 0\ns_cbranch_scc1 vm_none_%=\n"

// From the loop's head, or with `resume` from entry k for the lanes that wait for block `now`.
#define VM_STEPS(choose, none, B, N, R, T)                                                                                              \
    "s_getpc_b64 s[40:41]\nvm_here_%=:\ns_add_u32 s40, s40, vm_h0_%=-vm_here_%=\ns_addc_u32 s41, s41, 0\n"                  \
    "s_cmp_lg_u32 %[resume], 0\ns_cbranch_scc0 vm_head_%=\n"                                                                \
    "v_cmp_eq_u32 vcc, %[now], %[pc]\ns_mov_b64 exec, vcc\ns_cmp_eq_u32 %[resume], 1\ns_cbranch_scc1 vm_first_%=\n"        \
    "s_sub_u32 %[k], %[k], 1\n" B "s_add_u32 %[k], %[k], 1\ns_mov_b32 s46, s47\n" B                                         \
    "s_bitcmp1_b32 s46, 28\ns_cbranch_scc1 vm_push_%=\ns_branch vm_update_%=\n"                                            \
    "vm_head_%=:\n"                                                                                                         \
    "s_cmp_lt_i32 %[fuel], 1\ns_cbranch_scc1 vm_fuel_%=\nv_cmp_eq_u32 s[68:69], -16, %[pc]\n" choose                         \
    "s_cmp_lg_u64 s[68:69], 0\ns_cbranch_scc1 vm_idle_%=\n" none                                                            \
    "v_readlane_b32 %[k], %[record], s50\ns_and_b32 %[now], s50, 63\nv_cmp_eq_u32 vcc, %[now], %[pc]\n"                     \
    "s_lshr_b32 s52, %[k], 8\ns_sub_i32 %[fuel], %[fuel], s52\ns_bcnt1_i32_b64 %[count], vcc\n"                             \
    "s_mul_i32 s52, s52, %[count]\ns_add_u32 %[active], %[active], s52\ns_mov_b64 exec, vcc\n"                              \
    "vm_first_%=:\n"                                                                                                        \
    B "s_nop 0\n" N VM_HANDLERS(B, N, R)                                                      \
    VM_AT(34) T                                                                                                             \
    "vm_fuel_%=: s_mov_b32 %[event], 0\ns_branch vm_out_%=\n"                                                               \
    "vm_idle_%=: s_mov_b32 %[event], 1\ns_branch vm_out_%=\n"                                                               \
    "vm_none_%=: s_mov_b32 %[event], 2\ns_branch vm_out_%=\n"                                                               \
    "vm_modulo_%=: s_mov_b32 %[event], 4\ns_mov_b64 exec, -1\ns_branch vm_out_%=\n"                                         \
    "vm_rare_%=: s_mov_b32 %[event], 3\ns_mov_b64 exec, -1\n"                                                               \
    "vm_out_%=:\n"
enum : int { kOutOfFuel = 0, kIdle = 1, kNoneWaits = 2, kRareEntry = 3, kModulo = 4 };

// kWide: entries in two sets of registers.
template <bool kQueued, bool kMost, bool kWide>
__global__ __launch_bounds__(kWave* kWavesPerBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void pcvm_small_kernel(VmArgs va, SmallArgs sm)
{
    typedef unsigned long long u64;
    extern __shared__ __align__(16) unsigned char small_lds[];
    const int lane = threadIdx.x & (kWave - 1), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const long group = (long)blockIdx.x * kWavesPerBlock + w;
    // this lane's column in the stack arrays (queued runs: only lanes that take members have one)
    const long slot = kQueued ? group * sm.lanes + lane : group * kWave + lane;
    if (group * (kQueued ? sm.lanes : kWave) >= va.batch_pad) return;  // waves of the last workgroup beyond the last group
    const int W = sm.ring, depth = va.depth;
    // (a stack as deep as it may be has a full ring: low + W + 1 never exceeds the depth, if the ring has ever been full)
    const int full = min(W + 1, depth);
    u64* const rings = reinterpret_cast<u64*>(small_lds + (size_t)w * small_wave_bytes(sm.n_stacks, W)) + lane;
    typedef __attribute__((address_space(3))) unsigned char Lds;
    const unsigned base = (unsigned)(size_t)(Lds*)rings;
    const unsigned row_bytes = (unsigned)W * (8 * kWave), r_record = sm.tables->record[lane];
    const unsigned r_word = sm.tables->word[lane], r_lo = sm.tables->imm_lo[lane], r_hi = sm.tables->imm_hi[lane], r_row = sm.tables->stack[lane] * row_bytes;
    const int lane2 = kWide ? kWave + lane : lane;
    const unsigned r_word2 = sm.tables->word[lane2], r_lo2 = sm.tables->imm_lo[lane2], r_hi2 = sm.tables->imm_hi[lane2],
                   r_row2 = sm.tables->stack[lane2] * row_bytes;
    auto entry = [&](unsigned r, unsigned r2, int k) { return (unsigned)__builtin_amdgcn_readlane(kWide && (k & kWave) ? r2 : r, k & (kWave - 1)); };
    const unsigned input_stacks = sm.tables->input_stacks;
    file_own();

    // Queued runs: the first member of a lane is the one of its column, without asking; the queue holds those beyond the last
    // column.  (A lane that asks is one atomic of a wave on one address, and the fewer lanes a group has, the fewer ask
    // together: gcd, 20 000 members in 1000 groups, all members through the queue 0.225 ms, so 0.106; 313 full groups through the
    // queue, interpreter of larger programs, 0.178.)
    long member = slot;
    const bool valid = (!kQueued || lane < sm.lanes) && member < va.batch;
    // The code of the block a lane waits for, and the return addresses below it: the first pc_mem in memory, the next `held`
    // in f_hi, f_lo, the latest in the lowest bits.  held_max: how many of them there may be before memory, or the depth, is
    // reached.
    int pc = kRetired, held = 0, held_max = 0, pc_mem = 0;
    unsigned f_lo = 0, f_hi = 0;
    // Steps so far: `steps` of them up to the last look at the limit, since then as many as `fuel` is below `chunk`.
    const bool tracing = !kQueued && va.trace && group == 0;
    const int kChunk = tracing ? 1 : 1 << 20;
    long steps = 0, member_start = 0;
    int chunk = 0, fuel = 0;
    u64 active_steps = 0;
    unsigned active = 0;
    int my_error = 0;

    // "PUSH T onto x": a fresh execution has its inputs on the stacks, every other stack empty, and waits at block 0
    auto start_member = [&]() __attribute__((always_inline)) {
#pragma unroll 1
        for (int v = 0; v < va.n_vars; ++v)
            file_write((unsigned)v, v < va.n_inputs ? (u64)va.inputs[(size_t)v * va.batch + member] : 0ull, (input_stacks >> v) & 1u);
        pc = code_of(0);
        held = 0;
        pc_mem = 0;
        held_max = min(sm.frames, depth - 1);
        member_start = steps + (chunk - fuel);
    };
    if (valid) start_member();

    bool dry = va.batch_pad >= va.batch;  // queued runs: the queue is known to be empty
    int resume = 0, k = 0, now = 0, count = 0;
    const int lowest = code_of(va.n_blocks - 1);
    for (;;) {
        int event;
        auto scalar = [](auto& x) { x = __builtin_amdgcn_readfirstlane(x); };  // (which the compiler cannot know of an output)
        scalar(resume), scalar(k), scalar(now), scalar(fuel), scalar(active), scalar(count);
#define VM_OPERANDS                                                                                                         \
    : [pc] "+v"(pc), [held] "+v"(held), [f_lo] "+v"(f_lo), [f_hi] "+v"(f_hi), [k] "+s"(k), [now] "+s"(now),                 \
      [fuel] "+s"(fuel), [active] "+s"(active), [count] "+s"(count), [event] "=&s"(event)                                   \
    : [word] "v"(r_word), [lo] "v"(r_lo), [hi] "v"(r_hi), [row] "v"(r_row), [word2] "v"(r_word2), [lo2] "v"(r_lo2),         \
      [hi2] "v"(r_hi2), [row2] "v"(r_row2), [record] "v"(r_record), [base] "v"(base),                                       \
      [held_max] "v"(held_max), [mask] "s"(W - 1), [full] "s"(full), [lowest] "s"(lowest), [resume] "s"(resume),            \
      [f_down] "s"(sm.frame_bits), [f_up] "s"(32 - sm.frame_bits), [f_mask] "s"((1 << sm.frame_bits) - 1)                   \
    : "memory", "m0", "vcc", "scc", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", "s48", "s49", "s50", "s51", "s52",    \
      "s53", "s54", "s55", "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63", "s68", "s69"
#define VM_RUN(choose, none)                                                                                                \
    if constexpr (kWide)                                                                                                    \
        asm volatile(VM_STEPS(choose, none, VM_B2, VM_N2, VM_R2, VM_T2) VM_OPERANDS);                                              \
    else                                                                                                                    \
        asm volatile(VM_STEPS(choose, none, VM_B1, VM_N1, VM_R1, "") VM_OPERANDS)
        if constexpr (kMost) {
            VM_RUN(VM_CHOOSE_MOST, VM_NONE_MOST);
        } else if constexpr (kQueued) {
            VM_RUN(VM_CHOOSE_EARLIEST, VM_NONE_EARLIEST);
        } else {
            VM_RUN(VM_CHOOSE_EARLIEST "s_mov_b64 s[68:69], 0\n", VM_NONE_EARLIEST);
        }
#undef VM_RUN
#undef VM_OPERANDS
        scalar(event);
        resume = 0;
        if (event == kModulo) {  // (operands in v[116:119])
            unsigned al, ah, bl, bh;
            asm volatile("v_mov_b32 %0, v116\n\tv_mov_b32 %1, v117\n\tv_mov_b32 %2, v118\n\tv_mov_b32 %3, v119" : "=&v"(al), "=&v"(ah), "=&v"(bl), "=&v"(bh));
            const u64 a = (u64)al | (u64)ah << 32, b = (u64)bl | (u64)bh << 32, o = (b == 0 || b == ~0ull) ? 0ull : (u64)((long long)a % (long long)b);
            asm volatile("v_mov_b32 v116, %0\n\tv_mov_b32 v117, %1" ::"v"((unsigned)o), "v"((unsigned)(o >> 32)));
            resume = 2;
            continue;
        }
        if (event == kNoneWaits) break;
        if (event == kOutOfFuel) {
            if (tracing && chunk > 0 && lane == 0 && steps < va.trace_capacity) {  // (of the one step since the last look)
                va.trace[2 * steps] = code_of(now);
                va.trace[2 * steps + 1] = count;
            }
            steps += chunk - fuel;
            active_steps += active;
            active = 0;
            const long left = va.max_steps - steps;
            if (left <= 0) {
                if (!kQueued) {
                    if (__ballot(pc >= 0)) my_error = PCVM_E_STEP_LIMIT;
                    chunk = fuel = 0;
                    break;
                }
                if (pc >= 0 && steps - member_start >= va.max_steps) {  // this member does not halt: drop it
                    my_error = PCVM_E_STEP_LIMIT;
                    pc = kRetired;
                }
            }
            fuel = chunk = left <= 0 ? 1 : (int)min(left, (long)kChunk);
        } else if (event == kIdle) {
            const u64 before = __ballot(pc == kRetired);
            if (pc == kHalt) {
                const long next = dry ? va.batch : va.batch_pad + (long)atomicAdd(va.queue, 1ull);
                if (next < va.batch) {
                    member = next;
                    start_member();
                } else {
                    pc = kRetired;
                }
            }
            // (a lane that asked in vain: no other of the wave asks again.  200 000 members of gcd on 3072 groups, where 196 608
            // lanes would ask one address whether there are more: 0.76 -> 0.39 ms)
            dry = dry || __ballot(pc == kRetired) != before;
        } else {  // entry k - 1, with everything that can happen to it
            const unsigned word = entry(r_word, r_word2, k - 1), stack = entry(r_row, r_row2, k) / row_bytes;
            const int handler = (int)(word >> 24), row = (int)stack * W;
            const int half = sm.frames / 2, f_mask = (1 << sm.frame_bits) - 1;
            if (pc == now) {
                if (handler == kDoCall || handler == kDoCallJump) {
                    if (held + pc_mem >= depth - 1) {
                        my_error = min(my_error, (int)PCVM_E_STACK_OVERFLOW);
                    } else if (held >= held_max) {  // the registers are full: their earliest half makes room
                        const u64 frames = (u64)f_lo | (u64)f_hi << 32;
                        for (int q = 0; q < half; ++q)
                            va.pc_stacks[(size_t)(pc_mem + q) * va.batch_pad + slot] = (int)(frames >> (sm.frame_bits * (sm.frames - 1 - q))) & f_mask;
                        pc_mem += half;
                        held -= half;
                        held_max = min(sm.frames, depth - 1 - pc_mem);
                    }
                } else if (handler == kDoReturn) {
                    if (held <= 0 && pc_mem > 0) {
                        u64 frames = 0;
                        for (int q = 0; q < half; ++q)
                            frames = frames << sm.frame_bits | (u64)(unsigned)va.pc_stacks[(size_t)(pc_mem - half + q) * va.batch_pad + slot];
                        f_lo = (unsigned)frames;
                        f_hi = (unsigned)(frames >> 32);
                        pc_mem -= half;
                        held = half;
                        held_max = min(sm.frames, depth - 1 - pc_mem);
                    } else if (held <= 0) {
                        pc = kHalt;
                        if (kQueued) va.outputs[member] = (long long)file_read((unsigned)va.output_var);
                    }
                } else if (handler == kDoPop) {
                    unsigned c;
                    u64 x = file_read(word >> 8, c);
                    const int have = (int)(c & 0xffffu), low = (int)(c >> 16), idx = have - 2;  // entry that becomes the top
                    if (have <= 0) {
                        my_error = min(my_error, (int)PCVM_E_STACK_UNDERFLOW);
                    } else {
                        c -= 1;
                        if (idx >= 0 && idx < low) {  // below the ring
                            // (and with it as many as half the ring holds)
                            const int first = max(0, idx - W / 2);
                            const long long* const from = va.var_stacks + (size_t)stack * depth * va.batch_pad + slot;
                            x = (u64)from[(size_t)idx * va.batch_pad];
                            for (int q = first; q < idx; q += 4) {  // (four loads under way at a time)
                                u64 y[4];
#pragma unroll
                                for (int u = 0; u < 4; ++u) y[u] = (u64)from[(size_t)min(q + u, idx) * va.batch_pad];
#pragma unroll
                                for (int u = 0; u < 4; ++u)
                                    if (q + u < idx) rings[(row + ((q + u) & (W - 1))) * kWave] = y[u];
                            }
                            c = (unsigned)(have - 1) | (unsigned)first << 16;
                        } else if (idx >= 0) {
                            x = rings[(row + (idx & (W - 1))) * kWave];
                        }
                        file_write(word >> 8, x, c);
                    }
                } else {  // a push
                    unsigned c;
                    const u64 top = file_read(word >> 8, c);
                    const int have = (int)(c & 0xffffu), low = (int)(c >> 16);
                    if (have >= depth) {
                        my_error = min(my_error, (int)PCVM_E_STACK_OVERFLOW);
                    } else if (have - 1 - low >= W) {  // the ring is full: its lower half makes room
                        const int upto = min(low + max(1, W / 2), depth - W - 1);  // (see `full`)
                        long long* const to = va.var_stacks + (size_t)stack * depth * va.batch_pad + slot;
                        for (int q = low; q < upto; ++q) to[(size_t)q * va.batch_pad] = (long long)rings[(row + (q & (W - 1))) * kWave];
                        file_write(word >> 8, top, (unsigned)have | (unsigned)upto << 16);
                    }
                }
            }
            // (a push or a call that has room now, and a return with somewhere to go, run as if nothing had been)
            resume = 1;
            if (handler != kDoPop) k -= 1;
        }
        if (my_error && event == kRareEntry) pc = kRetired;  // a member in error stops; the others of its group go on
    }

    steps += chunk - fuel;
    active_steps += active;
    if (!kQueued && valid) va.outputs[member] = (long long)file_read((unsigned)va.output_var);
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
// of 3 lanes 10.2 ms, 47 of 64 lanes 12.1).  Beyond that groups are full, three per SIMD, which hide each other's latency in
// part (MOST_WAITING, one / two / three / four per SIMD: binomial, 10^6 members, 5.5 / 4.9 / 4.4 / 4.6 ms; collatz_steps, 200 000,
// 0.42 / 0.30 / 0.30 / 0.33; fibonacci, 200 000, 19.2 / 19.6 / 19.0 / 15.8).
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
    SmallTables tables;
    SmallArgs sm{};
    // (a limit that short runs can reach counts block by block)
    const bool most = queued && policy == PCVM_SCHED_MOST_WAITING;
    sm.n_stacks = pack_small(program, most && max_steps >= (1ll << 30), stack_depth, &tables);
    const bool small = sm.n_stacks >= 0;
    size_t small_lds = 0;
    void (*small_kernel)(VmArgs, SmallArgs) = nullptr;
    if (small) {
        int cus = 0, dev = 0;
        PCVM_TRY(hipGetDevice(&dev), PCVM_E_DEVICE);
        PCVM_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), PCVM_E_DEVICE);
        sm.frame_bits = 1;
        while ((1 << sm.frame_bits) < program->n_blocks) ++sm.frame_bits;
        sm.frames = 64 / sm.frame_bits;
        sm.lanes = kWave;
        if (queued) n_groups = queued_groups(batch, cus, &sm.lanes);
        // as long a ring as the workgroups of a compute unit can share its LDS for (up to four of them: the registers
        // allow no more to be useful)
        const long wgs = (n_groups + kWavesPerBlock - 1) / kWavesPerBlock;
        const long share = std::min<long>(4, (wgs + cus - 1) / cus);
        auto lds = [&](int ring) { return kWavesPerBlock * small_wave_bytes(sm.n_stacks, ring); };
        sm.ring = 1;
        while (sm.ring < stack_depth && lds(2 * sm.ring) <= (size_t)(kLdsBytes / share)) sm.ring *= 2;
        small_lds = lds(sm.ring);
        if (tables.n_entries <= kSmallMax)
            small_kernel = !queued ? pcvm_small_kernel<false, false, false> : most ? pcvm_small_kernel<true, true, false> : pcvm_small_kernel<true, false, false>;
        else
            small_kernel = !queued ? pcvm_small_kernel<false, false, true> : most ? pcvm_small_kernel<true, true, true> : pcvm_small_kernel<true, false, true>;
        PCVM_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(small_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes), PCVM_E_DEVICE);
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
    const bool deep_vars = !small || sm.ring < stack_depth, deep_pc = !small || sm.frames < stack_depth;
    const size_t var_bytes = deep_vars ? (size_t)(small ? sm.n_stacks : program->n_vars) * stack_depth * batch_pad * sizeof(long long) : 0;
    const size_t pc_bytes = deep_pc ? (size_t)stack_depth * batch_pad * sizeof(int) : 0;
    // (what is refused does not depend on how little of it a program really takes)
    const size_t lanes = (size_t)std::min<long>(n_groups * kWave, (long)((batch + kWave - 1) / kWave * kWave));
    const size_t largest = ((size_t)program->n_vars * sizeof(long long) + sizeof(int)) * stack_depth * lanes;
    if (largest > (size_t)64 << 30) return fail(PCVM_E_ALLOC, "stacks would need %zu bytes", largest);

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
    if (small)
        hipLaunchKernelGGL(small_kernel, dim3(blocks), dim3(kWave * kWavesPerBlock), small_lds, g_stream, va, sm);
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
