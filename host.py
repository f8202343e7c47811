import ctypes, sys, numpy as np
sys.path.insert(0,'/root/repo')
from perf import cases as C
N=ctypes.CDLL('./host_new.so'); O=ctypes.CDLL('./host_old.so')
for l in (N,O):
    l.refill_us.restype=l.estimate_us.restype=ctypes.c_double
P=[(c["name"],C._lengths(c),c["heads"],c["kv_heads"],c["head_dim"]) for c in C.listed() if c["path"]!="ring"]
P+=[("gqa",[3000,500],8,2,128),("long+short",[9000]+[100]*578,16,8,128),("d64",[16384],2,2,64),("many1",[64]*1000,32,4,128),("C5 2kv",[29082,18500,3311,2034]+[1500]*8,8,2,128)]
for name,L,hq,hkv,d in P:
    cu=(ctypes.c_int32*(len(L)+1))(*np.concatenate([[0],np.cumsum(L)]).astype(int).tolist())
    print('%-16s refill old %.1f new %.1f | estimate old %.1f new %.1f'%(name,O.refill_us(cu,len(L),hq,hkv,d,50),N.refill_us(cu,len(L),hq,hkv,d,50),O.estimate_us(cu,len(L),hq,hkv,d,30),N.estimate_us(cu,len(L),hq,hkv,d,30)))
